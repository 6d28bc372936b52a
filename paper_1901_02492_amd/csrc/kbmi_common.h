// Host helpers of the entry points and device helpers shared by the plane,
// top-k and filter translation units (not the search kernels).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstdint>

#include "kbmi_internal.h"

namespace kbmi {

kb_status launch_status(const char *what);

// Host helpers defined in kbmi_kernels.hip.
// Frame limits common to every kernel: 1 <= n_img <= 32767, h <= 2^30, w <= 2^27.
kb_status check_frame(int64_t n_img, int64_t h, int64_t w);
// Asynchronous host-to-device copy through a pinned staging buffer (the call
// does not wait for its stream).
kb_status staged_copy(void *dst, const void *src, size_t bytes, hipStream_t stream);
// Send tau_i = t_i - t_0 (double [n_img], at the workspace start) and the
// velocities (double2 [n_vel], at byte offset *vel_off, 16-byte aligned) to
// the workspace, for kernels that compute displacements on the device.
kb_status upload_tau_vel(const double *t, int64_t n_img, const double *vel, int64_t n_vel,
                         void *workspace, hipStream_t stream, size_t *vel_off);
// Send the gather table (planes of `pix_bytes` bytes per pair; velocities in
// visiting order unless visiting_order is false) and the visiting order to
// the workspace (workspace_layout offsets).
kb_status upload_table(const double *t, int64_t n_img, const double *vel, int64_t n_vel,
                       int64_t h, int64_t w, int64_t pix_bytes, void *workspace,
                       hipStream_t stream, bool visiting_order = true);

// Argument checks of kb_search (and its allocation-free variant).
kb_status check_search_args(const void *planes, int32_t dtype, const float *lp_scale,
                            int64_t n_img, int64_t h, int64_t w, const double *t,
                            const double *vel, int64_t n_vel, int64_t k_cand,
                            const void *cand_nu, const void *cand_alpha, const void *cand_vel,
                            const void *cand_nobs);
// Enqueue the search on checked arguments whose tables are already in
// `workspace` (workspace_layout offsets; the inverse scales of 16-bit planes
// are written here).
kb_status launch_search_in(const void *planes, int32_t dtype, const float *lp_scale,
                           int64_t n_img, int64_t h, int64_t w, int64_t n_vel, int64_t k_cand,
                           float *cand_nu, float *cand_alpha, int32_t *cand_vel,
                           int16_t *cand_nobs, void *workspace, const Reach &reach,
                           hipStream_t s);

// One displacement on the device: floor(v * tau + 0.5) as a separate IEEE
// double multiply, add and floor (no contraction), which rounds exactly as
// the host table does.  The conversion saturates to the int32 range.
__device__ inline int32_t displacement(double v, double tau) {
#pragma clang fp contract(off)
    const double f = floor(v * tau + 0.5);
    int32_t d;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(d) : "v"(f));
    return d;
}

// The pixel (index in its image) that start pixel (x0, y0) reaches at tau; ok
// says whether it is in the frame (index 0 if not).  Coordinates are added in
// 32 bits without a clamp: frames have at most 2^30 rows and 2^27 columns, so
// a saturated displacement lands outside [0, 2^31) or beyond the frame.  The
// FP64 and 64-bit integer instructions here are most of what the kernels that
// gather along candidates issue per image, hence no clamp and one wide
// multiply: 18 vector instructions for 40.  A step of 9 x 613 x 1187, 260
// velocities in bf16, re-scoring 52 a pixel: 3.00 -> 2.69 ms.
__device__ inline uint64_t displaced_pixel(double2 v, double tau, int x0, int y0, int h, int w,
                                           bool &ok) {
    const uint32_t x = (uint32_t)x0 + (uint32_t)displacement(v.x, tau);
    const uint32_t y = (uint32_t)y0 + (uint32_t)displacement(v.y, tau);
    ok = y < (uint32_t)h && x < (uint32_t)w;
    const uint64_t at = (uint64_t)y * (uint32_t)w + x;
    return ok ? at : 0;
}

// q / k for 0 <= q < 4096 and k >= 1, inv_k = 1.f / k: the quotient's distance
// from an integer above it is at least 1 / k, so half of that (q + 0.5)
// absorbs the rounding.
__device__ inline int small_quotient(int q, float inv_k) {
    return (int)(((float)q + 0.5f) * inv_k);
}

}  // namespace kbmi

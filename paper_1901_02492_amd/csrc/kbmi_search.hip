// Trajectory-search launchers for one plane format (KBMI_FMT: 0 = float32,
// 1 = IEEE half, 2 = bfloat16) and one group of list lengths (KBMI_GROUP);
// the build compiles this file once per (format, group).
#include <algorithm>

#include "kbmi_device.h"

#ifndef KBMI_FMT
#error "compile with -DKBMI_FMT=0|1|2"
#endif
#ifndef KBMI_GROUP
#error "compile with -DKBMI_GROUP=0..7"
#endif

namespace kbmi {
namespace {

TileMap tile_map(int w, int h) {
    TileMap tm;
    tm.nseg = (w + 63) / 64;
    tm.h = h;
    tm.strip = tm.nseg < KBMI_STRIP_TILES ? tm.nseg : KBMI_STRIP_TILES;
    tm.nblocks = tm.nseg * h;
    tm.sw = (KBMI_SUPER_W > 0 && tm.nseg % (8 * KBMI_SUPER_W) == 0) ? KBMI_SUPER_W : 0;
    return tm;
}

// Workgroups of the persistent grid for `Kernel` (0 if unknown): the number
// the device holds at once, at most KBMI_PERSIST_PER_CU per CU, cached per
// device and per kernel instance.  The cap keeps each XCD's block of start
// pixels small enough for its L2 when a short candidate list lets more waves
// fit.
template <auto Kernel>
int resident_workgroups() {
    static int cached[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if (cached[dev] == 0) {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, Kernel, 64, 0) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) !=
                hipSuccess)
            return 0;
        cached[dev] = std::min(per_cu, KBMI_PERSIST_PER_CU) * cus;
    }
    return cached[dev];
}

template <int KM>
kb_status launch_one(const StackView &v, hipStream_t s) {
    constexpr int PB = search_queue(KM, KBMI_FMT);
    // The persistent order pays for float32 planes; the 16-bit search keeps the
    // super-strip order, which measured faster (15 x 2048^2, 600 velocities, K = 50:
    // 14.1 ms against 17.6), except on long walks (kPaceVelocities).
    const bool long_walk = is_long_walk(v.n_img, v.n_vel, KBMI_FMT == KB_F32);
    if (KBMI_FMT == KB_F32 || (long_walk && search_waves(KM, KBMI_FMT) == 2)) {
        auto kernel = search_persistent_kernel<KM, PB, KBMI_FMT>;
        const int grid =
            resident_workgroups<search_persistent_kernel<KM, PB, KBMI_FMT>>();
        const int nseg = (v.w + 63) / 64;
        const int per_xcd = grid / 8;
        // Worth it only when the frame holds several generations of blocks.
        if (grid >= 8 && grid % 8 == 0 && per_xcd % KBMI_PERSIST_BS == 0 &&
            (int64_t)nseg * v.h >= 4 * (int64_t)grid) {
            PersistMap pm;
            pm.nseg = nseg;
            pm.h = v.h;
            pm.bs = KBMI_PERSIST_BS;
            pm.brows = per_xcd / KBMI_PERSIST_BS;
            pm.nbc = (nseg + pm.bs - 1) / pm.bs;
            pm.nbr = (v.h + pm.brows - 1) / pm.brows;
            pm.generations = block_generations(pm.nbc, pm.nbr);
            pm.spin = KBMI_PERSIST_SPIN;
            pm.long_walk = long_walk;
            hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(64), 0, s, v.sync, 8);
            kb_status st = launch_status("zero_words_kernel");
            if (st != KB_OK) return st;
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(64), 0, s, v.planes, v.inv_scale,
                               v.n_img, v.h, v.w, v.disp, v.disp_stride, v.vel_index, v.n_vel,
                               v.reach, v.k_cand, pm, v.cand_nu, v.cand_alpha, v.cand_vel,
                               v.cand_nobs, v.sync);
            return launch_status("search_persistent_kernel");
        }
    }
    const TileMap tm = tile_map(v.w, v.h);
    // Frames whose tiles leave waves idle: up to 8 waves share a tile's
    // velocities, as many as the device still holds at once (2048 waves), in
    // two chunks each so that waves with short and long chunks even out.  A
    // tile's wave otherwise waits for its own gathers only: 64 tiles, 121
    // velocities, K = 5: 82 us with 1 wave, 61 with 2, 49 with 4, 42 with 8; 300
    // tiles, 600 velocities, K = 50: 335, 239, 167, 176; 800 tiles, 3600 velocities,
    // 16-bit: 2070, 1430, 1640, 1770; 1255 tiles, 400 velocities: 279, 314, 297,
    // 385 (the merges of K = 50 lists and the shorter class runs cost more
    // than the idle waves).
    const int resident = resident_workgroups<search_kernel<KM, PB, KBMI_FMT>>();
    int parts = 1;
    while (parts < 8 && (int64_t)tm.nblocks * parts * 2 <= resident && v.n_vel >= 16 * parts &&
           search_split_lds_bytes<KM, PB>(2 * parts) <= kLdsBytes)
        parts *= 2;
    if (parts > 1) {
        const int chunk = std::min(kChunk, std::max(8, (v.n_vel + 2 * parts - 1) / (2 * parts)));
        hipLaunchKernelGGL((search_split_kernel<KM, PB, KBMI_FMT>), dim3(tm.nblocks),
                           dim3(64 * parts), (search_split_lds_bytes<KM, PB>(parts)), s, v.planes,
                           v.inv_scale, v.n_img, v.h, v.w, v.disp, v.disp_stride, v.vel_index,
                           v.n_vel, v.reach, v.k_cand, tm, chunk, v.cand_nu, v.cand_alpha,
                           v.cand_vel, v.cand_nobs);
        return launch_status("search_split_kernel");
    }
    hipLaunchKernelGGL((search_kernel<KM, PB, KBMI_FMT>), dim3(tm.nblocks), dim3(64), 0, s,
                       v.planes, v.inv_scale, v.n_img, v.h, v.w, v.disp, v.disp_stride,
                       v.vel_index, v.n_vel, v.reach, v.k_cand, tm, v.cand_nu, v.cand_alpha,
                       v.cand_vel, v.cand_nobs);
    return launch_status("search_kernel");
}

template <int KM>
kb_status launch_batch_km(const BatchJob *jobs, const BatchShape &b, int *resident,
                          hipStream_t s) {
    constexpr int PB = search_queue(KM, KBMI_FMT);
    auto kernel = search_batch_kernel<KM, PB, KBMI_FMT>;
    if (!jobs) {
        const int g = resident_workgroups<search_batch_kernel<KM, PB, KBMI_FMT>>();
        if (g < 8 || g % 8 != 0)
            return fail(KB_EDEVICE, "batched search: no persistent grid for this device (%d)", g);
        *resident = g;
        return KB_OK;
    }
    if (b.paced > 0) {
        hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(64), 0, s, b.sync, 8);
        const kb_status st = launch_status("zero_words_kernel");
        if (st != KB_OK) return st;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)b.grid), dim3(64), 0, s, jobs, b.n_jobs,
                       b.generations, b.paced, KBMI_PERSIST_SPIN, b.k_cand, b.sync);
    return launch_status("search_batch_kernel");
}

// List lengths of this translation unit's group are compiled; the others are
// left to their own units (the dispatcher never sends them here).
template <int K>
kb_status launch_in_group(const StackView &v, hipStream_t s) {
    if constexpr (km_group(K) == KBMI_GROUP) return launch_one<K>(v, s);
    else return fail(KB_EUNSUPPORTED, "list length %d is not compiled in this group", K);
}

template <int K>
kb_status launch_batch_in_group(const BatchJob *jobs, const BatchShape &b, int *resident,
                                hipStream_t s) {
    if constexpr (km_group(K) == KBMI_GROUP) return launch_batch_km<K>(jobs, b, resident, s);
    else return fail(KB_EUNSUPPORTED, "list length %d is not compiled in this group", K);
}

}  // namespace

template <>
kb_status launch_search_group<KBMI_FMT, KBMI_GROUP>(int km, const StackView &v, hipStream_t s) {
    switch (km) {
#define KB_CASE(K) \
    case K:        \
        return launch_in_group<K>(v, s);
        KB_SEARCH_KM_LIST(KB_CASE)
#undef KB_CASE
    }
    return fail(KB_EUNSUPPORTED, "k_cand above %d is not supported", KB_MAX_KCAND);
}

template <>
kb_status launch_search_batch_group<KBMI_FMT, KBMI_GROUP>(int km, const BatchJob *jobs,
                                                           const BatchShape &b, int *resident,
                                                           hipStream_t s) {
    switch (km) {
#define KB_CASE(K) \
    case K:        \
        return launch_batch_in_group<K>(jobs, b, resident, s);
        KB_SEARCH_KM_LIST(KB_CASE)
#undef KB_CASE
    }
    return fail(KB_EUNSUPPORTED, "k_cand above %d is not supported", KB_MAX_KCAND);
}

}  // namespace kbmi

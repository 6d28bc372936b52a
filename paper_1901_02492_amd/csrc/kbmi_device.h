// Device-side building blocks of libkbmi shared by its translation units:
// raw buffer access, candidate keys, the start-pixel tile order, and the
// trajectory-search kernels (instantiated per plane format by kbmi_search.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <utility>

#include "kbmi_internal.h"
#include "kbmi_merge_network.h"

// Launch-shape defaults (compile-time tunables).
#ifndef KBMI_STRIP_TILES
#define KBMI_STRIP_TILES 4      // start-pixel tiles per strip of the tile order
#endif
#ifndef KBMI_PATCH_TILES
#define KBMI_PATCH_TILES 64     // consecutive tiles of the strip order that one XCD takes
#endif
#ifndef KBMI_SUPER_W
#define KBMI_SUPER_W 2          // tiles per XCD strip in the super-strip order (0: off)
#endif
#ifndef KBMI_SUPER_ROWS
#define KBMI_SUPER_ROWS 64      // rows after which the XCDs change strips in that order
#endif
#ifndef KBMI_PERSIST_BS
#define KBMI_PERSIST_BS 2       // float32 planes: tiles per block row in the persistent order
#endif
#ifndef KBMI_PERSIST_SPIN
#define KBMI_PERSIST_SPIN 4000  // bound of a wave's wait at a generation boundary
#endif
#ifndef KBMI_PERSIST_PER_CU
#define KBMI_PERSIST_PER_CU 8   // persistent grid: at most this many one-wave workgroups per CU
#endif
// List lengths compiled for the search (each slot costs registers and
// compare-and-swap work on every insertion); a search keeps k_cand
// candidates in the shortest compiled list of at least k_cand slots, which
// gives the same best k_cand.  Every length in this list must be in
// kKmList below, in the same order.
#define KB_SEARCH_KM_LIST(X)                                                                \
    X(2) X(4) X(6) X(8) X(12) X(16) X(20) X(24) X(28) X(32) X(36) X(40) X(44) X(48) X(50) \
    X(52) X(56) X(60) X(64)

namespace kbmi {

// One search problem as the host launchers see it.
struct StackView {
    const void *planes;        // [n_img][h][w] (psi, phi) pairs of the plane format
    const float2 *inv_scale;   // 16-bit planes: (1/s_psi, 1/s_phi) per image, padded with 0
    int n_img, h, w;
    const GatherEntry *disp;   // gather-table rows in visiting order, `disp_stride` entries each
    int disp_stride;
    const int32_t *vel_index;  // original index of each visited velocity
    int n_vel, k_cand;
    Reach reach;
    float *cand_nu, *cand_alpha;
    int32_t *cand_vel;
    int16_t *cand_nobs;
    uint32_t *sync;            // per-XCD generation counters of the persistent search
};

// One stack of a batched search, as the batch kernel reads it from device
// memory.  The launch's work items are its jobs' tiles: job j owns items
// [item_begin_j, item_begin_{j+1}), item_begin a multiple of 8.  A dense job's
// items are its tiles in strip order; a block job starts at a generation
// boundary and its items are the paced persistent order of a single-stack
// search (generation (item - item_begin) / grid, workgroup
// (item - item_begin) % grid), slots past its frame's edge included and
// skipped.
struct BatchJob {
    const void *planes;
    const float2 *inv_scale;
    const GatherEntry *disp;
    const int32_t *vel_index;
    float *cand_nu, *cand_alpha;
    int32_t *cand_vel;
    int16_t *cand_nobs;
    int n_img, h, w, disp_stride, n_vel;
    int item_begin;
    int nseg;                  // tiles per row
    int dense;                 // 1: strip order (strip tiles wide); 0: block order
    int strip;
    int bs, brows, nbc, nbr;   // block order (PersistMap's fields)
    int long_walk;
    Reach reach;
};

// The launch of a batch: `grid` workgroups, `generations` generations, the
// first `paced` of them paced through `sync`.
struct BatchShape {
    int n_jobs, k_cand;
    int grid, generations, paced;
    uint32_t *sync;
};

// Waves of a search kernel per SIMD.  16-bit planes take as many as a short list
// leaves registers for, two batches of 16 loads and 16 images' scales beside it
// (12 x 2048^2 f16, 600 velocities, K = 5 11.6 ms with 2 waves, 8.3 with 3, 7.0 with 4).
// One more spills: K = 10 with 4 waves 11.3 ms for 8.7 with 3, in bfloat16, whose
// values take two registers more to widen, 15.1 for 9.4.
// Float32 planes, whose gathers keep the memory path busy with two, lose as
// much by the shorter queue: 20 x 500 x 900, K = 10 2.14 ms with 2, 2.19 with 3, 2.43 with 4.
constexpr int search_waves(int km, int fmt) {
    return fmt == KB_F32 || km > 20 ? 2 : km <= (fmt == KB_F16 ? 8 : 6) ? 4 : 3;
}
// Queued candidates per lane before a merge: as many as that many waves' queues
// and lists leave room for in a CU's LDS, which is given out in pieces of 1280
// bytes (a queue of 14 takes 11 and leaves room for 11 waves, one of 13 takes 10 and
// leaves 12: 8 x 1024^2 f16, 600 velocities, K = 10 2.12 -> 1.92 ms).  A merge takes 16;
// with a queue of 22 more of them are filled when one of the wave's lanes runs
// full (K = 50, 16 -> 22: 12 x 251 x 301, 400 velocities 0.291 -> 0.281 ms;
// 25 x 1024 x 2048 f16, 4000 velocities 75.2 -> 74.3 ms).
constexpr int search_queue(int km, int fmt) {
    return search_waves(km, fmt) == 4 ? 9 : search_waves(km, fmt) == 3 ? 13 : 22;
}

kb_status launch_status(const char *what);

// Search launchers.  km is the (even) compiled list length >= k_cand.  The
// list lengths are split into kKmGroups groups, km in group (km / 2 - 1) %
// kKmGroups, and the build compiles kbmi_search.hip once per plane format and
// group (the translation units compile in parallel); launch_search and
// launch_search_batch dispatch to them.
constexpr int kKmGroups = 8;
constexpr int kKmList[] = {2, 4, 6, 8, 12, 16, 20, 24, 28, 32, 36, 40, 44, 48, 50, 52, 56, 60, 64};
constexpr int kKmCount = (int)(sizeof(kKmList) / sizeof(kKmList[0]));
static_assert(kKmList[kKmCount - 1] == KB_MAX_KCAND, "the longest list is KB_MAX_KCAND");
constexpr int km_index(int km) {
    for (int i = 0; i < kKmCount; ++i)
        if (kKmList[i] == km) return i;
    return -1;
}
constexpr int km_group(int km) { return km_index(km) % kKmGroups; }
// The compiled list length for k_cand (1 <= k_cand <= KB_MAX_KCAND).
constexpr int km_for(int k_cand) {
    for (int i = 0; i < kKmCount; ++i)
        if (kKmList[i] >= k_cand) return kKmList[i];
    return -1;
}
template <int FMT, int G>
kb_status launch_search_group(int km, const StackView &v, hipStream_t s);
template <int FMT, int G>
kb_status launch_search_batch_group(int km, const BatchJob *jobs, const BatchShape &b,
                                    int *resident, hipStream_t s);
#define KBMI_DECLARE_GROUP(F, G)                                                          \
    template <>                                                                           \
    kb_status launch_search_group<F, G>(int, const StackView &, hipStream_t);             \
    template <>                                                                           \
    kb_status launch_search_batch_group<F, G>(int, const BatchJob *, const BatchShape &,    \
                                              int *, hipStream_t);
#define KBMI_DECLARE_FMT(F)                                                                 \
    KBMI_DECLARE_GROUP(F, 0) KBMI_DECLARE_GROUP(F, 1) KBMI_DECLARE_GROUP(F, 2)             \
    KBMI_DECLARE_GROUP(F, 3) KBMI_DECLARE_GROUP(F, 4) KBMI_DECLARE_GROUP(F, 5)             \
    KBMI_DECLARE_GROUP(F, 6) KBMI_DECLARE_GROUP(F, 7)
KBMI_DECLARE_FMT(0)
KBMI_DECLARE_FMT(1)
KBMI_DECLARE_FMT(2)
#undef KBMI_DECLARE_FMT
#undef KBMI_DECLARE_GROUP
kb_status launch_search(int fmt, int km, const StackView &v, hipStream_t s);
// One launch over the jobs of a batch.  With jobs == nullptr nothing is
// launched and *resident receives the workgroups the device holds at once.
kb_status launch_search_batch(int fmt, int km, const BatchJob *jobs, const BatchShape &b,
                              int *resident, hipStream_t s);

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// The gather table, the visiting order and the inverse scales do not change
// during a launch: they are read through the constant address space, so
// their wave-uniform loads stay scalar whatever else the kernel writes.
typedef __attribute__((address_space(4))) const i32x4 const_i32x4;
typedef __attribute__((address_space(4))) const f32x4 const_f32x4;
typedef __attribute__((address_space(4))) const int32_t const_i32;

// Raw buffer loads with the descriptor as four plain words.
__device__ u32x2 raw_load_b64(i32x4 rsrc, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.load.v2i32");
__device__ uint32_t raw_load_b32(i32x4 rsrc, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.load.i32");

namespace {

// ---------------------------------------------------------------------------
// Raw buffer access.  A descriptor is four scalar words: the 48-bit base
// address, the record count in bytes (stride 0: an access is out of range when
// its byte offset is >= the record count, and then a load returns 0 without
// touching memory), and the format word.  The loads take the descriptor as a
// plain vector so that building one costs no masking.
// ---------------------------------------------------------------------------
constexpr int kBufferFlags = 0x00020000;


__device__ inline i32x4 buffer_words(uint64_t base, uint32_t bytes) {
    i32x4 r;
    r.x = (int)(uint32_t)base;
    r.y = (int)(uint32_t)(base >> 32);
    r.z = (int)bytes;
    r.w = kBufferFlags;
    return r;
}

// ---------------------------------------------------------------------------
// Candidate keys.  A candidate is ordered by (nu descending, j ascending); the
// 63-bit key (order-preserving bits of nu) << 31 | (0xFFFF - j) << 15 | n_obs
// compares the same way as unsigned integers.  n_obs never decides an order
// because j is unique within a pixel.  Key 0 is below every real candidate
// (nu = -inf maps to 0x007FFFFF) and marks an empty slot.
//
// Read as an IEEE double, such a key is non-negative (bit 63 is clear) and
// finite (the order bits are clamped to those of +inf, so the exponent field
// never reaches all ones), and doubles of that kind order exactly like their
// bit patterns: the FP64 max/min instructions move a key in one instruction.
// ---------------------------------------------------------------------------
__device__ inline uint32_t nu_order_bits(float nu) {
    uint32_t u = __float_as_uint(nu);
    if (u == 0x80000000u) u = 0u;   // -0 ranks equal to +0
    const uint32_t o = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return min(o, 0xFF800000u);     // nothing ranks above +inf
}

__device__ inline float nu_from_order_bits(uint32_t o) {
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}

__device__ inline uint64_t make_key(float nu, int j, uint32_t nobs) {
    return ((uint64_t)nu_order_bits(nu) << 31) |
           (uint64_t)(((uint32_t)(0xFFFF - j) << 15) | (nobs & 0x7FFFu));
}
__device__ inline float key_nu(uint64_t k) { return nu_from_order_bits((uint32_t)(k >> 31)); }
__device__ inline int32_t key_vel(uint64_t k) {
    return 0xFFFF - (int32_t)((uint32_t)(k >> 15) & 0xFFFFu);
}
__device__ inline int32_t key_nobs(uint64_t k) { return (int32_t)((uint32_t)k & 0x7FFFu); }

// k, n <- max(k, n), min(k, n) as keys, in place.
__device__ inline void key_exchange(uint64_t &k, uint64_t &n) {
    double kd = __builtin_bit_cast(double, k), t;
    asm("v_min_f64 %0, %1, %2\n\tv_max_f64 %1, %1, %2"
        : "=&v"(t), "+v"(kd)
        : "v"(__builtin_bit_cast(double, n)));
    k = __builtin_bit_cast(uint64_t, kd);
    n = __builtin_bit_cast(uint64_t, t);
}

// k <- max(k, n) as keys.
__device__ inline uint64_t key_max(uint64_t k, uint64_t n) {
    double kd = __builtin_bit_cast(double, k);
    asm("v_max_f64 %0, %0, %1" : "+v"(kd) : "v"(__builtin_bit_cast(double, n)));
    return __builtin_bit_cast(uint64_t, kd);
}

// Merging a batch of 16 queued candidates into the descending list of KM
// (registers 0..KM-1 of r/ra; the batch in KM..KM+15) with the generated
// comparator network, keeping the best KM.  Alpha follows its key.
template <int KIND, int A, int B, int N>
__device__ __forceinline__ void net_op(uint64_t (&r)[N], float (&ra)[N]) {
    const bool c = r[B] > r[A];
    if constexpr (KIND == 0) {
        key_exchange(r[A], r[B]);
        const float t = c ? ra[B] : ra[A];
        ra[B] = c ? ra[A] : ra[B];
        ra[A] = t;
        // Materialise both outputs here (no code): otherwise the alpha
        // selects sink to their uses and every compare result stays live.
        asm volatile("" : "+v"(r[A]), "+v"(r[B]), "+v"(ra[A]), "+v"(ra[B]));
    } else {
        r[A] = key_max(r[A], r[B]);
        ra[A] = c ? ra[B] : ra[A];
        asm volatile("" : "+v"(r[A]), "+v"(ra[A]));
    }
}
template <int KM, int N, size_t... I>
__device__ __forceinline__ void net_run(uint64_t (&r)[N], float (&ra)[N],
                                        std::index_sequence<I...>) {
    // Applied in program order: interleaving the network's independent
    // exchanges would only lengthen live ranges past the register file.
    ((net_op<MergeNetwork<KM>::ops[I].kind, MergeNetwork<KM>::ops[I].a,
             MergeNetwork<KM>::ops[I].b>(r, ra),
      __builtin_amdgcn_sched_barrier(0)),
     ...);
}
template <int KM, int N, size_t... S>
__device__ __forceinline__ void net_place(uint64_t (&r)[N], float (&ra)[N],
                                          std::index_sequence<S...>) {
    // List slot s takes register perm[s] (fixed swaps of the network).
    const uint64_t k[KM] = {r[MergeNetwork<KM>::perm[S]]...};
    const float a[KM] = {ra[MergeNetwork<KM>::perm[S]]...};
    ((r[S] = k[S], ra[S] = a[S]), ...);
}
template <int KM, int N>
__device__ __forceinline__ void net_merge(uint64_t (&r)[N], float (&ra)[N]) {
    net_run<KM>(r, ra, std::make_index_sequence<MergeNetwork<KM>::n_ops>());
    net_place<KM>(r, ra, std::make_index_sequence<KM>());
}

// Sorts slots [LO, LO + N) descending where they fall and then rise (bitonic,
// any N: the power of two goes last).
template <int LO, int N, int KR>
__device__ __forceinline__ void sort_valley(uint64_t (&key)[KR], float (&al)[KR]) {
    if constexpr (N > 1) {
        constexpr int M = N > 32 ? 32 : N > 16 ? 16 : N > 8 ? 8 : N > 4 ? 4 : N > 2 ? 2 : 1;
#pragma unroll
        for (int i = LO; i < LO + N - M; ++i) {
            const uint64_t a = key[i], b = key[i + M];
            const float fa = al[i], fb = al[i + M];
            const bool c = b > a;
            key[i] = c ? b : a;
            key[i + M] = c ? a : b;
            al[i] = c ? fb : fa;
            al[i + M] = c ? fa : fb;
        }
        sort_valley<LO, N - M>(key, al);
        sort_valley<LO + N - M, M>(key, al);
    }
}

// Scores of one trajectory (Sec. 2.1.5): nu = Psi / sqrt(Phi) and
// alpha = Psi / Phi; Phi = 0 (no valid observation) gives nu = -inf and
// alpha = 0.  Every kernel scores with these functions, so equal sums give
// bitwise equal scores.
// KBMI_IEEE_SCORE 0: both from the hardware reciprocal square root r of Phi
// (within 1 ulp for normal inputs; Phi below 2^-100 is scaled by 2^64 first,
// so no denormal reaches it): nu = Psi * r, alpha = nu * r.
// KBMI_IEEE_SCORE 1: a correctly rounded square root and divisions.
#ifndef KBMI_IEEE_SCORE
#define KBMI_IEEE_SCORE 0
#endif
__device__ inline float inv_sqrt_phi(float F) {
    if (KBMI_IEEE_SCORE) return 0.f;
    const bool tiny = F < 0x1p-100f;
    const float r = __builtin_amdgcn_rsqf(tiny ? F * 0x1p64f : F);
    return tiny ? r * 0x1p32f : r;
}
__device__ inline float score_nu(float P, float F, float r) {
    if (KBMI_IEEE_SCORE) return F > 0.f ? P / sqrtf(F) : -INFINITY;
    return F > 0.f ? P * r : -INFINITY;
}
__device__ inline float score_alpha(float P, float nu, float F, float r) {
    if (KBMI_IEEE_SCORE) return F > 0.f ? P / F : 0.f;
    (void)P;
    return F > 0.f ? nu * r : 0.f;
}

// Start-pixel tiles: one wave = 64 adjacent pixels of one row.  Tiles are
// enumerated in strips `strip` tiles wide (all rows of a strip, then the next
// strip) so that consecutive workgroups cover a compact 2-D patch, and the
// workgroup index is remapped so that each of the 8 XCDs (which receive
// workgroups round-robin) takes KBMI_PATCH_TILES consecutive tiles of that
// order (one patch, whose gathers share its L2) at a time.  The patches go
// round the XCDs because a tile's work is the images its trajectories stay in,
// which changes across the frame: with one contiguous range each, the launch
// waited for the XCD of the left-most columns (12 x 251 x 301, 400 velocities: 0.314
// -> 0.300 ms).
__device__ inline int xcd_remap(int b, int nblocks) {
    const int xcd = b & 7, k = b >> 3;
    constexpr int P = KBMI_PATCH_TILES;
    const int full = nblocks / (8 * P) * (8 * P);
    if (b < full) return (k / P * 8 + xcd) * P + k % P;
    // The rest of the order: one contiguous range each.
    const int q = (nblocks - full) >> 3, r = (nblocks - full) & 7;
    return full + xcd * q + (xcd < r ? xcd : r) + (k - (full >> 3));
}

__device__ inline void strip_tile(int t, int nseg, int h, int strip, int &row, int &seg) {
    const int fs = nseg / strip;
    const int full = fs * h * strip;
    if (t < full) {
        const int s = t / (h * strip);
        const int rem = t - s * h * strip;
        row = rem / strip;
        seg = s * strip + (rem - (rem / strip) * strip);
    } else {
        const int rw = nseg - fs * strip;
        const int rem = t - full;
        row = rem / rw;
        seg = fs * strip + (rem - (rem / rw) * rw);
    }
}

// Super-strip order (used when nseg is a multiple of 8 * sw): the frame is
// cut into vertical super-strips 8 * sw tiles wide; the eight XCDs sweep down
// one together, each in one of its sw-tile strips, so the rows that later
// start rows gather again (every velocity reaches up to the longest
// displacement) stay within a window the memory-side cache can hold.  Every
// KBMI_SUPER_ROWS rows each XCD moves one strip to the right, so that none
// keeps the columns whose trajectories see the most images (25 x 1024 x 2048 f16,
// 4000 velocities: 88.4 -> 76.0 ms).
__device__ inline void superstrip_tile(int b, int h, int sw, int &row, int &seg) {
    const int xcd = b & 7, m = b >> 3;
    const int per = sw * h;
    const int ss = m / per;
    const int rem = m - ss * per;
    row = rem / sw;
    seg = (ss * 8 + ((xcd + row / KBMI_SUPER_ROWS) & 7)) * sw + (rem - row * sw);
}

struct TileMap {
    int nseg;     // tiles per row
    int h;        // rows
    int strip;    // tiles per strip
    int nblocks;  // nseg * h
    int sw;       // > 0: super-strip order with sw-tile strips per XCD

    __device__ inline void map(int b, int &row, int &seg) const {
        if (sw > 0) superstrip_tile(b, h, sw, row, seg);
        else strip_tile(xcd_remap(b, nblocks), nseg, h, strip, row, seg);
    }
};

// Persistent order: the grid is exactly the number of workgroups the GPU
// holds at once, and workgroup w processes one tile per generation.  In a
// generation, XCD x (workgroups w = 8k + x, dispatched round-robin over the
// XCDs) covers one block of bs x brows tiles (k -> row k / bs, seg k % bs).
// The eight XCDs take eight side-by-side blocks and generations move down the
// frame, then to the next eight block columns (the last columns, fewer than
// eight, are taken row by row, eight blocks a generation).  Waves that start
// a generation together walk the velocities roughly in step, so one
// velocity's gathers find the rows the block read for the previous ones
// still in L2.  The XCDs change columns every generation: a block's work
// falls with the images its trajectories still see, and an XCD that kept the
// first column had up to 1.5 times the others' (13 x 1024^2, 32000 velocities:
// 186 -> 167 ms).  Every in-frame tile belongs to exactly one (generation,
// workgroup); slots past the frame's edge are skipped.
inline __host__ __device__ int block_generations(int nbc, int nbr) {
    return (nbc >> 3) * nbr + ((nbc & 7) * nbr + 7) / 8;
}
struct PersistMap {
    int nseg, h;
    int bs, brows;     // block: bs tiles wide, brows rows tall (bs * brows = grid / 8)
    int nbc, nbr;      // blocks per row of blocks, rows of blocks
    int generations;   // block_generations(nbc, nbr)
    int spin;          // bound of a wave's wait at a generation boundary (0: no wait)
    int long_walk;     // 1: also wait after every kPaceVelocities velocities
    __device__ inline bool map(int gen, int w, int &row, int &seg) const {
        const int xcd = w & 7, k = w >> 3;
        const int sc = min(gen / nbr, nbc >> 3);
        const int wide = min(8, nbc - 8 * sc);
        const int g = gen - sc * nbr;
        const int id = 8 * g + ((xcd + g) & 7);
        const int br = id / wide, bc = 8 * sc + id - br * wide;
        const int q = k / bs;
        row = br * brows + q;
        seg = bc * bs + (k - q * bs);
        return br < nbr && row < h && seg < nseg;
    }
};

template <int FMT>
struct PlaneLoad {                       // one (psi, phi) pair as loaded
    typedef u32x2 type;                  // float32: two words
};
template <>
struct PlaneLoad<KB_F16> {
    typedef uint32_t type;               // 16-bit: psi low half, phi high half
};
template <>
struct PlaneLoad<KB_BF16> {
    typedef uint32_t type;
};

__device__ inline float lp_value(uint32_t bits16, int fmt) {
    if (fmt == KB_F16) return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
    return __uint_as_float(bits16 << 16);
}

// ---------------------------------------------------------------------------
// Trajectory search.
//
// One wave (one workgroup) owns 64 adjacent start pixels of one row and walks
// every velocity.  Per velocity each lane gathers its trajectory's (psi, phi)
// pairs (one coalesced 512-byte run per image across the wave), sums them in
// image order and scores nu.
//
// What bounds it.  The vector-memory path returns a wave's 8-byte load in
// 16.4 cycles and its 4-byte load in 10.7, whether it hits, misses the frame
// or finds a zero-length buffer; with a load per image that path is busy 93 %
// of the time (13 x 1024^2, 32000 velocities: 1.336e11 of 1.436e11 cycles), the
// vector issue 37 %.  So the loads that read nothing are the cost to remove.  A
// linear trajectory that leaves the frame does not return (displacements
// grow with the image in both axes), so a tile sees a velocity in a prefix
// 1 .. m of the images: the velocities are sorted into classes by m, a chunk
// at a time, and each class is visited by a loop with exactly its number of
// loads, rounded up to even (class_of), so that the wait before a batch's sums counts the
// loads behind it (a branch around single loads makes the compiler wait for
// all: 25 images, float32, 902 -> 1655 ms).  m comes from a binary search in
// the table's own displacements, a velocity per lane.  A load per image ->
// classes and balanced tile orders: 13 x 1024^2, 32000 velocities, K = 50
// 237 -> 165 ms (15.0 -> 8.9 loads a velocity); 12 x 251 x 301, 400 velocities 0.374 ->
// 0.281; 25 x 1024 x 2048 f16, 4000 velocities, K = 50 79.8 -> 65.9 (kPaceVelocities);
// 25 x 1500^2, 1000 velocities, K = 50 46.3 -> 22.3; 9 x 613 x 1187 bf16,
// 260 velocities, K = 52 1.50 -> 1.21; 15 x 4096^2, 600 velocities, K = 50 (12.8 of 14
// images seen) 79.5 -> 80.0, bound by the same path at 20 cycles a load, most
// of them from L2.  Images and velocities keep their order within a class; the
// sums of a velocity run in image order and the selection does not depend on
// the order of the velocities, so results are bit for bit those of any order.
//
// Per-pixel selection keeps a descending list of KM >= k_cand keys in
// registers.  Inserting into it costs a compare-and-swap per slot, and the wave
// pays for it whenever any lane inserts, so candidates are first filtered
// against a per-lane threshold (the list's last key at the last merge) and
// parked in a per-lane LDS queue of PB entries; the queue is merged into the
// list only when some lane's queue is full (and at the end).  A candidate that
// fails the threshold can never enter the final list: the threshold only rises.
// The merge stands once, outside the class loops (in each of them the list
// would be copied at every loop's edge and spill: 4x slower): a loop leaves
// when a queue is full, and its gathers in flight are issued again after the
// merge.
//
// The list's registers bound the kernel to two to four waves per SIMD
// (search_waves): memory-level parallelism comes from the waves, each with two
// batches' gathers in flight.
// ---------------------------------------------------------------------------
constexpr int kChunk = 256;           // velocities classified at once
// Velocities between two paces inside a tile of a long walk.  Tiles that see
// fewer images run ahead of the others of their XCD's block, and with more
// images than 17 an XCD's L2 holds hardly more than one velocity's windows
// (24 displaced images: 3.1 MB of 4), so over thousands of velocities the block
// falls apart: 25 x 4096^2, 4000 velocities, float32 1521 ms with the generation's
// pace alone, 714 with one every 1024 velocities too (903 without classes, in
// step by themselves); 25 x 2048 x 4096, 3000 velocities 284 -> 266.  Fewer images
// lose by the waiting (13 x 1024^2, 32000 velocities, every 512: 186 -> 228).
// 16-bit planes with lists for two waves a SIMD walk in the paced order then:
// 25 x 1024 x 2048, 4000 velocities 73.8 -> 65.9 ms, 25 x 4096^2 757 -> 608, 25 x 2048 x 4096,
// 3000 velocities 272 -> 228.  The line lies at 18 images; K = 50, unpaced / paced:
// 2048^2, 4000 velocities, float32 17 images 115 / 119 ms, 18 134 / 136, 20 138 / 138, 25
// 163 / 158; f16 15 images 72 / 84, 18 130 / 128; 25 x 4096^2 f16, 2400 velocities 423 / 387.
// Shorter 16-bit lists, with more waves, lose by that order: 20 x 2048^2 f16, 4000
// velocities, K = 20 97 / 148, K = 10 99 / 146.
constexpr int kPaceVelocities = 1024;
static_assert(kPaceVelocities % kChunk == 0, "a pace stands between two chunks");
constexpr int kMaxScaleImages = 64;   // 16-bit planes: images whose inverse scales lie in the LDS
inline bool is_long_walk(int64_t n_img, int64_t n_vel, bool f32) {
    return n_img > 17 && n_vel >= 2 * kPaceVelocities && (f32 || n_img <= kMaxScaleImages);
}
constexpr int kHeldScaleWords = 2 * kMaxScaleImages + 2 * 16;
constexpr int kScaleWords = kHeldScaleWords + 2 * 16;   // and those of one batch of later images
// LDS words of visit_velocities: a chunk's list and classes, then the inverse
// scales of 16-bit planes.
constexpr int kVisitWords = kChunk + kChunk / 2 + kChunk / 4 + kScaleWords;

// LDS of a search workgroup: the candidate queue (3 words per entry and
// lane), also used to stage the output (KM words per lane), then the words of
// visit_velocities.
template <int KM, int PB>
constexpr int search_queue_words() {
    return (3 * PB > KM ? 3 * PB : KM) * 64;
}
template <int KM, int PB>
constexpr int search_lds_words() {
    return search_queue_words<KM, PB>() + kVisitWords;
}

__device__ inline int wave_lane() { return (int)threadIdx.x & 63; }
// Orders one wave's LDS accesses (a workgroup may hold waves that are
// elsewhere): the LDS serves a wave in order, so this only binds the compiler.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sums of one pixel along one trajectory.
template <int FMT>
struct PixelSums {
    float P = 0.f, F = 0.f;
    uint32_t c = 0u;
    // float32 planes: psi, phi as loaded.
    __device__ inline void add(u32x2 v) {
        uint32_t m;
        P += __uint_as_float(v.x);
        F += __uint_as_float(v.y);
        // n_obs: the stored phi is nonzero exactly at valid pixels.
        // min(bits, 1) as one vector instruction: the compiler's
        // compare-and-carry form routes each term through a scalar mask and
        // needs wait states before its use.
        asm("v_min_u32 %0, %1, 1" : "=v"(m) : "v"(v.y));
        c += m;
    }
    // 16-bit planes: the packed pair and its image's inverse scales, exact
    // powers of two (the product is exact, so each FMA rounds once).
    __device__ inline void add(uint32_t v, float isp, float isf) {
        uint32_t m;
        P = fmaf(lp_value(v & 0xFFFFu, FMT), isp, P);
        F = fmaf(lp_value(v >> 16, FMT), isf, F);
        // Both halves at once: min(psi16, 1) | min(phi16, 1) << 16; at most
        // 32767 terms, so the low half never carries.
        asm("v_pk_min_u16 %0, %1, %2" : "=v"(m) : "v"(v), "v"(0x00010001u));
        c += m;
    }
    __device__ inline uint32_t count() const { return FMT == KB_F32 ? c : c >> 16; }
};

// A tile (64 start pixels of one row, from column seg * 64 on) and what its
// gathers share.  All members but x and start are wave-uniform.
template <int FMT>
struct Tile {
    typedef typename PlaneLoad<FMT>::type LoadT;
    static constexpr uint32_t kPix = FMT == KB_F32 ? 8u : 4u;   // bytes per (psi, phi) pair
    uint64_t row0;          // address of the start row in image 0
    uint32_t row_bytes;
    const GatherEntry *disp;
    int stride, n_img, h, row;
    const const_i32 *visit;
    uint32_t *list;         // LDS: velocities of the class being visited
    uint16_t *seen;         // LDS: images a velocity is visible in, image 0 apart
    uint8_t *cls;           // LDS: its class
    float *scale;           // LDS: inverse scales, image i at 2 (i - 1), up to kMaxScaleImages
    const float *more_scale;   // the same of all images, in memory
    int x;                  // this lane's start column
    PixelSums<FMT> start;   // its pixel's sums in image 0

    // Inverse scales of the images from i on (0-based after image 0), nv of them.
    __device__ inline const float *scales(int i, int nv) const {
        if (i + nv <= kMaxScaleImages) return scale + 2 * i;
        float *own = scale + kHeldScaleWords;
        const int q = wave_lane();
        if (q < 2 * nv) own[q] = i + q / 2 < n_img - 1 ? more_scale[2 * i + q] : 0.f;
        wave_sync();
        return own;
    }
    __device__ inline LoadT load(uint64_t base, uint32_t bytes, int dx) const {
        const i32x4 rs = buffer_words(base, bytes);
        if constexpr (FMT == KB_F32) return raw_load_b64(rs, (x + dx) * (int)kPix, 0, 0);
        else return raw_load_b32(rs, (x + dx) * (int)kPix, 0, 0);
    }
};

// The entries of a list from the q-th on; q stops at the last.  A list in LDS is
// held an entry by each lane; with `run` not 0 it is run + 0, run + 1, ..
struct ListCursor {
    const uint32_t *list;
    int n, q;
    uint32_t run, held;
    __device__ inline ListCursor(const uint32_t *l, uint32_t r, int count, int from)
        : list(l), n(count), q(from), run(r), held(0) {
        if (run == 0) load();
    }
    __device__ inline void load() { held = list[min((q & ~63) + wave_lane(), n - 1)]; }
    __device__ inline uint32_t entry() const {
        if (run != 0) return run + (uint32_t)q;
        return (uint32_t)__builtin_amdgcn_readlane((int)held, q & 63);
    }
    __device__ inline void step() {
        if (q + 1 < n) {
            ++q;
            if (run == 0 && (q & 63) == 0) load();
        }
    }
};

enum { kOne, kMany, kManyMore };

// The velocities of the class in t.list (with RUNS: or of the run, if not 0) from
// the q-th on, n of them: calls finish(j, P, F, n_obs) for each with the
// velocity's original index j and the sums of this lane's pixel, until full()
// (the selection's queue may not hold two more) or the list ends; returns the
// next q.
//   NV     loads of a batch.  Where a velocity of an even class sees one image
//          less, the last load is not real: a zero-length buffer, whose base is
//          never dereferenced
//   PARTS  batches of a velocity: one; several, of images whose scales the LDS
//          holds; several, also of later images
// Two batches are in flight: the gathers of the next are issued before the
// current one is summed and scored, and the table entries of the one after are
// fetched behind them, into the registers the next one's just left.  Rows of
// the displaced window are in the frame for every real load, columns are cut by
// the buffer's range check.  Fetched entries may pass the end of the table by
// up to 14 (the order array lies there); their loads are not real.
template <int NV, int PARTS, int FMT, bool RUNS, class Finish, class Full>
__device__ __forceinline__ int visit_class(const Tile<FMT> &t, int v0, uint32_t run_, int n,
                                           int q, Finish &&finish, Full &&full) {
    typedef typename Tile<FMT>::LoadT LoadT;
    constexpr bool MULTI = PARTS != kOne;
    q = __builtin_amdgcn_readfirstlane(q);   // (uniform: said again where it is lost)
    n = __builtin_amdgcn_readfirstlane(n);
    const uint32_t run = RUNS ? __builtin_amdgcn_readfirstlane(run_) : 0u;
    ListCursor cur(t.list, run, n, q);
    // The entries in e: those of velocity `place` of the chunk, part part_f of
    // parts_f, of which left_f are visible.
    int part_f = 0, parts_f = 1, left_f = 0, j_f = 0;
    const const_i32x4 *row_f = nullptr;
    auto enter = [&]() {
        const uint32_t ent = cur.entry();
        const int place = v0 + (int)(ent & 0xFFFFu);
        left_f = (int)(ent >> 16);
        part_f = 0;
        if constexpr (MULTI) parts_f = (left_f + NV - 1) / NV;
        row_f = (const const_i32x4 *)(const void *)(t.disp + (size_t)place * t.stride + 1);
        j_f = t.visit[place];
    };
    auto fetch = [&](i32x4(&e)[NV]) {
#pragma unroll
        for (int b = 0; b < NV; ++b) e[b] = row_f[b];
    };
    auto advance = [&]() {
        if (MULTI && ++part_f < parts_f) {
            row_f += NV;
            left_f -= NV;
        } else {
            cur.step();
            enter();
        }
    };
    auto issue = [&](const i32x4(&e)[NV], LoadT(&v)[NV]) {
#pragma unroll
        for (int b = 0; b < NV; ++b) {
            const uint64_t off = ((uint64_t)(uint32_t)e[b].w << 32) | (uint32_t)e[b].z;
            const bool real = (MULTI || (NV % 2 == 0 && b == NV - 1)) ? b < left_f : true;
            v[b] = t.load(t.row0 + off, real ? t.row_bytes : 0u, e[b].x);
        }
    };
    // 16-bit planes: the inverse scales of one batch's images stay in vector
    // registers.  (Read from the LDS for each velocity they would make its sums
    // wait for the entries just fetched, which the scalar path returns in any
    // order: 12 x 4096^2 f16, 600 velocities, K = 50 54.9 -> 51.5 ms.)
    constexpr bool kHeld = FMT != KB_F32 && !MULTI;
    float held[2 * NV];
    if constexpr (kHeld) {
#pragma unroll
        for (int b = 0; b < 2 * NV; ++b) {
            held[b] = t.scale[b];
            asm volatile("" : "+v"(held[b]));
        }
    }
    i32x4 e[NV];
    LoadT va[NV], vb[NV];
    enter();
    fetch(e);
    issue(e, va);
    int j_c = j_f, parts_c = parts_f;    // of the velocity being summed
    advance();
    fetch(e);
    PixelSums<FMT> sum = t.start;
    int part = 0;
    auto step = [&](LoadT(&cur_v)[NV], LoadT(&ahead)[NV]) {
        issue(e, ahead);
        const int j_a = j_f, parts_a = parts_f;
        __builtin_amdgcn_sched_barrier(0);
        advance();
        fetch(e);
        __builtin_amdgcn_sched_barrier(0);
        const float *sc = nullptr;
        if constexpr (PARTS == kManyMore) sc = t.scales(NV * part, NV);
        else if constexpr (FMT != KB_F32) sc = t.scale + 2 * (NV * part);
#pragma unroll
        for (int b = 0; b < NV; ++b) {
            if constexpr (FMT == KB_F32) {
                sum.add(cur_v[b]);
            } else if constexpr (kHeld) {
                sum.add(cur_v[b], held[2 * b], held[2 * b + 1]);
            } else {
                sum.add(cur_v[b], sc[2 * b], sc[2 * b + 1]);
            }
        }
        if (!MULTI || ++part == parts_c) {
            part = 0;
            if (q < n) finish(j_c, sum.P, sum.F, sum.count());
            ++q;
            sum = t.start;
        }
        j_c = j_a;
        parts_c = parts_a;
    };
    // Two batches a turn with one way out (an exit between them would cost the
    // compiler its scalar registers): at most two velocities end between two
    // chances to leave.  A velocity left in the middle is started again.
    do {
        step(va, vb);
        step(vb, va);
    } while (q < n && !full());
    return min(q, n);
}

#define KB_BATCH_LIST(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(10) X(12) X(14) X(16)

// The class of m visible images of `all`: the loads of its batch, or kMulti and
// those of each of several.  One batch's loads are rounded up to even, so that
// a frame whose edges cut trajectories has half the classes to begin anew, but
// for the velocities that all of up to 8 images see: on large frames these are
// most, and a load in 8 is worth it (8 x 4096^2 float32, 600 velocities, K = 5 49.5 ->
// 46.5 ms; exact classes throughout: 12 x 300^2, K = 5 0.421 -> 0.437 ms).
constexpr int kMulti = 15;
template <int MAXNV>
__device__ inline int class_of(int m, int all) {
    const int parts = (m + MAXNV - 1) / MAXNV;
    if (parts > 1) return kMulti + ((m + parts - 1) / parts + 1) / 2 * 2;
    return m == all && m <= 8 ? m : (m + 1) / 2 * 2;
}

// The velocities of one tile (start row `row`, start columns seg*64 ..
// seg*64+63) that wave `part` of `parts` takes, every parts-th chunk of
// `chunk` (at most kChunk) velocities: calls finish(j, P, F, n_obs) with the
// velocity's original index j and the sums of this lane's pixel, and drain()
// where full(), and pace() after every kPaceVelocities velocities.  All scalar
// arguments are wave-uniform.  words: kVisitWords of LDS; MAXNV: loads of a
// batch, at most.
template <int FMT, int MAXNV, bool RUNS, class Finish, class Full, class Drain, class Pace>
__device__ __forceinline__ void visit_velocities(
    uint32_t *words, const void *__restrict__ planes, const float2 *__restrict__ inv_scale,
    int n_img, int h, int w, const GatherEntry *__restrict__ disp, int disp_stride,
    const int32_t *__restrict__ vel_index, int n_vel, const Reach &reach, int row, int seg,
    int part, int parts, int chunk, Finish &&finish, Full &&full, Drain &&drain, Pace &&pace) {
    const int lane = wave_lane();
    Tile<FMT> t;
    t.row_bytes = (uint32_t)w * Tile<FMT>::kPix;
    t.row0 = reinterpret_cast<uint64_t>(planes) + (uint64_t)row * t.row_bytes;
    t.disp = disp;
    t.stride = disp_stride;
    t.n_img = n_img;
    t.h = h;
    t.row = row;
    const int x_first = seg * 64, x_last = min(seg * 64 + 63, w - 1);
    t.visit = (const const_i32 *)(const void *)vel_index;
    t.list = words;
    t.seen = reinterpret_cast<uint16_t *>(words + kChunk);
    t.cls = reinterpret_cast<uint8_t *>(words + kChunk + kChunk / 2);
    float *scale = reinterpret_cast<float *>(words + kChunk + kChunk / 2 + kChunk / 4);
    t.scale = scale;
    t.x = x_first + lane;
    if constexpr (FMT != KB_F32) {
        // Image 1 first (0 past the last image: a gather there reads 0).
        const float *isc = reinterpret_cast<const float *>(inv_scale + 1);
        for (int q = lane; q < kHeldScaleWords; q += 64)
            scale[q] = q < 2 * n_img - 2 ? isc[q] : 0.f;
        t.more_scale = isc;
        wave_sync();
    }
    // Image 0 is the start image: its displacement is (0, 0) for every
    // velocity (tau_0 = 0), so its pair is loaded once per tile and every
    // trajectory's sums start from it, 0 + value first.
    {
        const auto v0 = t.load(t.row0, t.row_bytes, 0);
        if constexpr (FMT == KB_F32) t.start.add(v0);
        else t.start.add(v0, inv_scale[0].x, inv_scale[0].y);
    }
    const int ni = n_img - 1;
    // A tile that no trajectory leaves sees every velocity in every image: one
    // class, in order, with no list and no look at the table, of which every
    // lane reads a line of its own.  (16-bit planes and large float32 frames, with
    // lists that leave registers for it: 15 x 2048^2 f16, 600 velocities, K = 10 9.95 -> 9.3
    // ms; 8 x 2048^2 float32, K = 1 12.2 -> 11.2.  Small float32 frames have few such
    // tiles and lose 1 to 2 % by the question: 12 x 251 x 301, K = 5.)
    const bool inside = RUNS && ni > 0 && row + reach.y_lo >= 0 && row + reach.y_hi < h &&
                        x_last + reach.x_lo >= 0 && x_first + reach.x_hi < w;
    const uint32_t run = inside ? (uint32_t)ni << 16 : 0u;
    if (inside && parts == 1) chunk = kPaceVelocities;
    for (int v0 = part * chunk; v0 < n_vel; v0 += parts * chunk) {
        if (v0 > 0 && v0 % kPaceVelocities == 0) pace();
        const int nc = min(chunk, n_vel - v0);
        uint32_t present = inside ? 1u << class_of<MAXNV>(ni, ni) : 0u;   // the chunk's classes
        if (!inside) {
            for (int k0 = 0; k0 < nc; k0 += 64) {
                const int k = k0 + lane;
                const GatherEntry *entries = disp + (size_t)(v0 + min(k, nc - 1)) * disp_stride;
                auto visible = [&](int i) {
                    const int dx = entries[i].dx, dy = entries[i].dy;
                    return (unsigned)(row + dy) < (unsigned)h && x_last + dx >= 0 &&
                           x_first + dx < w;
                };
                int m = ni, out = ni;
                if (ni > 0 && !visible(ni)) m = 0;
                while (__any(out - m > 1)) {
                    const int i = (m + out) >> 1;
                    const bool see = visible(i);
                    if (out - m > 1) (see ? m : out) = i;
                }
                const int c = class_of<MAXNV>(m, ni);
                t.seen[k] = (uint16_t)m;
                t.cls[k] = (uint8_t)c;
                uint64_t todo = __ballot(k < nc);
                while (todo != 0) {
                    const int c0 = __builtin_amdgcn_readlane(c, __builtin_ctzll(todo));
                    present |= 1u << c0;
                    todo &= ~__ballot(c == c0);
                }
            }
        }
        while (present != 0) {
            const int c0 = __builtin_ctz(present);
            present &= present - 1;
            int n = inside ? nc : 0;
            for (int k0 = 0; k0 < nc && !inside; k0 += 64) {
                const int k = k0 + lane;
                const bool hit = k < nc && t.cls[k] == c0;
                const uint64_t b = __ballot(hit);
                if (hit)
                    t.list[n + __builtin_amdgcn_mbcnt_hi(
                                   (uint32_t)(b >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0))] =
                        (uint32_t)k | ((uint32_t)t.seen[k] << 16);
                n += __builtin_popcountll(b);
            }
            wave_sync();
            for (int q = 0; q < n;) {
                if (c0 == 0) {
                    do {
                        const int k =
                            __builtin_amdgcn_readfirstlane((int)(t.list[q++] & 0xFFFFu));
                        finish(t.visit[v0 + k], t.start.P, t.start.F, t.start.count());
                    } while (q < n && !full());
                }
#define KB_CASE(NV)                                                                          \
    if constexpr (NV <= MAXNV) {                                                             \
        if (c0 == NV) q = visit_class<NV, kOne, FMT, RUNS>(t, v0, run, n, q, finish, full);  \
    }                                                                                        \
    if constexpr (NV % 2 == 0 && NV <= MAXNV && NV > MAXNV / 2) {                            \
        if (c0 == kMulti + NV) {                                                             \
            if (FMT == KB_F32 || n_img - 1 <= kMaxScaleImages)                               \
                q = visit_class<NV, kMany, FMT, RUNS>(t, v0, run, n, q, finish, full);       \
            else if constexpr (FMT != KB_F32)                                                \
                q = visit_class<NV, kManyMore, FMT, RUNS>(t, v0, run, n, q, finish, full);   \
        }                                                                                    \
    }
                KB_BATCH_LIST(KB_CASE)
#undef KB_CASE
                if (full()) drain();
            }
            wave_sync();
        }
    }
}

// The search of one tile (start row `row`, start columns seg*64 .. seg*64+63)
// by a workgroup of `parts` waves (a power of two), of which this is wave
// `part`.  lds: search_lds_words for each wave (and parts / 2 lists, for
// several).  All scalar arguments are wave-uniform.
template <int KM, int PB, int FMT, bool RUNS, class Pace>
__device__ __forceinline__ void search_tile(
    Pace &&pace, uint32_t *group_lds, int part, int parts, int chunk,
    const void *__restrict__ planes, const float2 *__restrict__ inv_scale,
    int n_img, int h, int w, const GatherEntry *__restrict__ disp, int disp_stride,
    const int32_t *__restrict__ vel_index, int n_vel, const Reach &reach, int k_cand, int row,
    int seg, float *__restrict__ cand_nu, float *__restrict__ cand_alpha,
    int32_t *__restrict__ cand_vel, int16_t *__restrict__ cand_nobs) {
    uint32_t *lds = group_lds + part * search_lds_words<KM, PB>();
    uint32_t *q_hi = lds;
    uint32_t *q_lo = lds + PB * 64;
    float *q_al = reinterpret_cast<float *>(lds + 2 * PB * 64);

    const int lane = wave_lane();

    // The list (slots 0..KM-1, descending); with the network merge, slots
    // KM..KM+15 receive the queued batch during a merge.
    constexpr int kBatch = 16;   // queued candidates a network merge takes
    constexpr bool kNet = KM >= 16;
    constexpr int KR = kNet ? KM + kBatch : KM;
    uint64_t key[KR];
    float al[KR];
#pragma unroll
    for (int s = 0; s < KR; ++s) {
        key[s] = 0;
        al[s] = 0.f;
    }
    uint64_t thr = 0;   // admission threshold (list tail at the last merge)
    int nq = 0;         // queued candidates of this lane

    // One pass of the insertion network: slot s keeps the larger key, the
    // smaller moves on (keys within a pixel are distinct, so one compare
    // decides where alpha goes).
    auto insert = [&](uint64_t nk, float a) {
#pragma unroll
        for (int s = 0; s < KM; ++s) {
            const bool c = nk > key[s];
            key_exchange(key[s], nk);
            const float ta = c ? al[s] : a;
            al[s] = c ? a : al[s];
            a = ta;
        }
    };
    auto merge_queue = [&]() {
        if constexpr (kNet) {
            // The lane's queue (entries past nq read as empty) into the batch
            // slots, then one network merge.  What a lane has queued beyond a
            // batch moves to the front.
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int at = (b < PB ? b : 0) * 64 + lane;
                const bool queued = b < PB && b < nq;
                const uint64_t nk = ((uint64_t)q_hi[at] << 32) | q_lo[at];
                const float na = q_al[at];
                key[KM + b] = queued ? nk : 0;
                al[KM + b] = queued ? na : 0.f;
            }
            net_merge<KM>(key, al);
#pragma unroll
            for (int b = kBatch; b < PB; ++b) {
                q_hi[(b - kBatch) * 64 + lane] = q_hi[b * 64 + lane];
                q_lo[(b - kBatch) * 64 + lane] = q_lo[b * 64 + lane];
                q_al[(b - kBatch) * 64 + lane] = q_al[b * 64 + lane];
            }
            nq = nq > kBatch ? nq - kBatch : 0;
        } else {
            for (int b = 0; b < PB; ++b) {
                if (!__any(b < nq)) break;
                if (b < nq) {
                    const uint64_t nk =
                        ((uint64_t)q_hi[b * 64 + lane] << 32) | q_lo[b * 64 + lane];
                    if (nk > key[KM - 1]) insert(nk, q_al[b * 64 + lane]);
                }
            }
            nq = 0;
        }
        thr = key[KM - 1];
    };
    // Score one trajectory (Sec. 2.1.5: nu = Psi / sqrt(Phi), alpha = Psi / Phi)
    // and queue it if it beats the admission threshold.  n_obs sits in the
    // low bits of the key and never decides an order.
    auto finish = [&](int j, float P, float F, uint32_t c) {
        const float r = inv_sqrt_phi(F);
        const float nu = score_nu(P, F, r);
        const uint64_t nk = make_key(nu, j, 0u);
        if (nk > thr) {
            q_hi[nq * 64 + lane] = (uint32_t)(nk >> 32);
            q_lo[nq * 64 + lane] = (uint32_t)nk | c;
            q_al[nq * 64 + lane] = score_alpha(P, nu, F, r);
            ++nq;
        }
    };
    // At most two velocities end before it is asked again.
    auto full = [&]() { return __any(nq >= PB - 1) != 0; };

    // Loads of a batch: two batches lie beside the list.  16-bit planes, 25
    // images, K = 50: 16 / 12 / 8 loads 73.8 / 77.0 / 87.9 ms.  Lists of 52 and more
    // spill with 16, but a limit below costs more where images fill a batch of 16
    // (K = 52, 600 velocities, 16 / 14 loads: 16 x 2048^2 f16 14.4 / 18.9 ms, 17 x
    // 2048^2 14.6 / 19.5, 15 x 2048^2 13.7 / 13.5, bfloat16 15.5 / 14.9).  Float32: K = 52
    // to 64 in batches of 8.
    constexpr int kMaxNv = KM <= 50 || FMT != KB_F32 ? 16 : 8;
    constexpr bool kRuns = RUNS && 3 * KM + 4 * kMaxNv <= 200;   // (K <= 44)
    visit_velocities<FMT, kMaxNv, kRuns>(lds + search_queue_words<KM, PB>(), planes, inv_scale,
                                         n_img, h, w, disp, disp_stride, vel_index, n_vel, reach,
                                         row, seg, part, parts, chunk, finish, full, merge_queue,
                                         pace);
    do merge_queue();
    while (__any(nq > 0));

    // Several waves: the upper half hands its lists to the lower half until
    // one is left.  Of two descending lists the larger of slot s and slot
    // KM - 1 - s are the best KM, falling and then rising.
    if (parts > 1) {
        for (int half = parts >> 1; half > 0; half >>= 1) {
            __syncthreads();   // the LDS is free of queues and of earlier lists
            uint32_t *slot = group_lds + (part < half ? part : part - half) * (3 * KM * 64) + lane;
            if (part >= half && part < 2 * half) {
#pragma unroll
                for (int s = 0; s < KM; ++s) {
                    slot[(3 * s) * 64] = (uint32_t)(key[s] >> 32);
                    slot[(3 * s + 1) * 64] = (uint32_t)key[s];
                    slot[(3 * s + 2) * 64] = __float_as_uint(al[s]);
                }
            }
            __syncthreads();
            if (part < half) {
#pragma unroll
                for (int s = 0; s < KM; ++s) {
                    const int o = KM - 1 - s;
                    const uint64_t k =
                        ((uint64_t)slot[(3 * o) * 64] << 32) | slot[(3 * o + 1) * 64];
                    const float a = __uint_as_float(slot[(3 * o + 2) * 64]);
                    const bool c = k > key[s];
                    key[s] = c ? k : key[s];
                    al[s] = c ? a : al[s];
                }
                sort_valley<0, KM>(key, al);
            }
        }
        if (part != 0) return;
    }

    // Write the rank-ordered list: stage each field through LDS so that the
    // wave's stores cover the contiguous [pixels][k_cand] run of its pixels
    // (one pixel's k_cand <= 64 entries per store instruction).
    const int npx = (w - seg * 64) < 64 ? (w - seg * 64) : 64;
    const size_t base = ((size_t)row * (size_t)w + (size_t)seg * 64) * (size_t)k_cand;
    wave_sync();
#pragma unroll
    for (int field = 0; field < 4; ++field) {
#pragma unroll
        for (int s = 0; s < KM; ++s) {
            uint32_t v;
            if (field == 0) v = __float_as_uint(key_nu(key[s]));
            else if (field == 1) v = __float_as_uint(al[s]);
            else if (field == 2) v = (uint32_t)key_vel(key[s]);
            else v = (uint32_t)key_nobs(key[s]);
            lds[lane * KM + s] = v;
        }
        wave_sync();
        if (lane < k_cand) {
            for (int p = 0; p < npx; ++p) {
                const uint32_t v = lds[p * KM + lane];
                const size_t o = base + (size_t)p * (size_t)k_cand + (size_t)lane;
                if (field == 0) cand_nu[o] = __uint_as_float(v);
                else if (field == 1) cand_alpha[o] = __uint_as_float(v);
                else if (field == 2) cand_vel[o] = (int32_t)v;
                else cand_nobs[o] = (int16_t)v;
            }
        }
        wave_sync();
    }
}

template <int KM, int PB, int FMT>
__global__ __launch_bounds__(64, search_waves(KM, FMT)) void search_kernel(
    const void *__restrict__ planes, const float2 *__restrict__ inv_scale, int n_img, int h,
    int w, const GatherEntry *__restrict__ disp, int disp_stride,
    const int32_t *__restrict__ vel_index,
    int n_vel, Reach reach, int k_cand, TileMap tiles, float *__restrict__ cand_nu,
    float *__restrict__ cand_alpha, int32_t *__restrict__ cand_vel,
    int16_t *__restrict__ cand_nobs) {
    auto pace = []() {};
    __shared__ __align__(16) uint32_t lds[search_lds_words<KM, PB>()];
    int row, seg;
    tiles.map(blockIdx.x, row, seg);
    search_tile<KM, PB, FMT, (FMT != KB_F32)>(
        pace, lds, 0, 1, kChunk, planes, inv_scale, n_img, h, w, disp, disp_stride, vel_index,
        n_vel, reach, k_cand, row, seg, cand_nu, cand_alpha, cand_vel, cand_nobs);
}

// The single-stack search of frames with too few tiles to fill the GPU: the
// workgroup's waves share a tile's velocities.
constexpr size_t kLdsBytes = 160 * 1024;   // of a CU
template <int KM, int PB>
constexpr size_t search_split_lds_bytes(int parts) {
    const size_t a = (size_t)parts * search_lds_words<KM, PB>() * 4;
    const size_t b = (size_t)(parts / 2) * 3 * KM * 64 * 4;
    return a > b ? a : b;
}
template <int KM, int PB, int FMT>
__global__ __launch_bounds__(512, 2) void search_split_kernel(
    const void *__restrict__ planes, const float2 *__restrict__ inv_scale, int n_img, int h,
    int w, const GatherEntry *__restrict__ disp, int disp_stride,
    const int32_t *__restrict__ vel_index, int n_vel, Reach reach, int k_cand, TileMap tiles,
    int chunk,
    float *__restrict__ cand_nu, float *__restrict__ cand_alpha, int32_t *__restrict__ cand_vel,
    int16_t *__restrict__ cand_nobs) {
    auto pace = []() {};
    extern __shared__ __align__(16) uint32_t split_lds[];
    int row, seg;
    tiles.map(blockIdx.x, row, seg);
    const int part = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    search_tile<KM, PB, FMT, false>(pace, split_lds, part, (int)blockDim.x >> 6, chunk, planes,
                                    inv_scale, n_img, h, w, disp, disp_stride, vel_index, n_vel,
                                    reach, k_cand, row, seg, cand_nu, cand_alpha, cand_vel,
                                    cand_nobs);
}

// The pacing of one XCD's workgroups.  The wait only shapes timing; no result
// depends on it.
struct XcdPace {
    uint32_t *count;    // arrivals of this XCD
    uint32_t per_xcd, target;
    int spin;           // bound of a wait; 0 once one has timed out (the XCD's
                        // workgroups are not all resident, e.g. beside another launch)
    __device__ inline XcdPace(uint32_t *sync, int s)
        : count(sync + (blockIdx.x & 7)), per_xcd(gridDim.x >> 3), target(0), spin(s) {}
    // This workgroup is n paces further; then wait (a bounded time) until every
    // workgroup of the XCD is, so that its waves go on together.
    __device__ inline void pace(int n) {
        if (threadIdx.x == 0)
            __hip_atomic_fetch_add(count, (uint32_t)n, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        target += (uint32_t)n * per_xcd;
        int i = 0;
        for (; i < spin; ++i) {
            if (__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= target)
                break;
            __builtin_amdgcn_s_sleep(8);
        }
        if (i == spin) spin = 0;
    }
};
// Paces inside a tile of a long walk.
__device__ inline int paces_inside(int n_vel) { return (n_vel - 1) / kPaceVelocities; }

// The single-stack search in the persistent order (large frames).
template <int KM, int PB, int FMT>
__global__ __launch_bounds__(64, search_waves(KM, FMT)) void search_persistent_kernel(
    const void *__restrict__ planes, const float2 *__restrict__ inv_scale, int n_img, int h,
    int w, const GatherEntry *__restrict__ disp, int disp_stride,
    const int32_t *__restrict__ vel_index, int n_vel, Reach reach, int k_cand, PersistMap pm,
    float *__restrict__ cand_nu, float *__restrict__ cand_alpha, int32_t *__restrict__ cand_vel,
    int16_t *__restrict__ cand_nobs, uint32_t *sync) {
    __shared__ __align__(16) uint32_t lds[search_lds_words<KM, PB>()];
    XcdPace xcd(sync, pm.spin);
    auto pace = [&]() {
        if (pm.long_walk) xcd.pace(1);
    };
    for (int gen = 0; gen < pm.generations; ++gen) {
        int row, seg;
        const bool ok = pm.map(gen, (int)blockIdx.x, row, seg);
        if (ok)
            search_tile<KM, PB, FMT, true>(pace, lds, 0, 1, kChunk, planes, inv_scale, n_img, h, w,
                                           disp, disp_stride, vel_index, n_vel, reach, k_cand, row,
                                           seg, cand_nu, cand_alpha, cand_vel, cand_nobs);
        // Generation boundary.
        xcd.pace(ok || !pm.long_walk ? 1 : 1 + paces_inside(n_vel));
    }
}

__global__ void zero_words_kernel(uint32_t *p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0u;
}

// ---------------------------------------------------------------------------
// Batched search: one launch covers the tiles of several stacks (the serving
// path), whatever their image counts.  In generation g, workgroup w processes
// work item g * grid + w (see BatchJob); after the first `paced` generations,
// which hold the jobs in block order, it waits with the others of its XCD as
// in the single-stack persistent search.  Without such jobs there is one
// generation of one workgroup per tile (batch_grid), so that the hardware balances
// tiles of unlike work; the jobs with the longest tiles come first.  (One launch per
// image-count class, each with its own tail, took 1.80 ms for six stacks of 5
// to 20 images and up to 400 x 500 pixels; one launch takes 0.92 ms.)  Each tile runs exactly the
// single-stack search, so a stack's results do not depend on what it is
// batched with.
// ---------------------------------------------------------------------------
template <int KM, int PB, int FMT>
__global__ __launch_bounds__(64, search_waves(KM, FMT)) void search_batch_kernel(
    const BatchJob *__restrict__ jobs_, int n_jobs, int generations, int paced, int spin,
    int k_cand, uint32_t *sync) {
    __shared__ __align__(16) uint32_t lds[search_lds_words<KM, PB>()];
    // The descriptors do not change during the launch: read through the
    // constant address space, their fields stay in scalar registers.
    typedef __attribute__((address_space(4))) const BatchJob CJob;
    const CJob *jobs = (const CJob *)(const void *)jobs_;
    const int grid = (int)gridDim.x;
    // A block job fills its generations, so that every workgroup waits as often.
    XcdPace xcd(sync, spin);
    for (int gen = 0; gen < generations; ++gen) {
        const int item = gen * grid + (int)blockIdx.x;
        int j = 0;
        for (int end = n_jobs; end - j > 1;) {   // the last job that begins at or before item
            const int mid = (j + end) >> 1;
            if (item >= jobs[mid].item_begin) j = mid;
            else end = mid;
        }
        const CJob &jb = jobs[j];
        const int li = item - jb.item_begin;
        int row = 0, seg = 0;
        bool ok;
        if (jb.dense) {
            ok = li < jb.nseg * jb.h;
            if (ok) strip_tile(xcd_remap(li, jb.nseg * jb.h), jb.nseg, jb.h, jb.strip, row, seg);
        } else {
            PersistMap pm;
            pm.nseg = jb.nseg;
            pm.h = jb.h;
            pm.bs = jb.bs;
            pm.brows = jb.brows;
            pm.nbc = jb.nbc;
            pm.nbr = jb.nbr;
            const int gl = li / grid;
            ok = gl < block_generations(jb.nbc, jb.nbr) && pm.map(gl, li - gl * grid, row, seg);
        }
        const Reach reach{jb.reach.x_lo, jb.reach.x_hi, jb.reach.y_lo, jb.reach.y_hi};
        const bool walk = gen < paced && jb.long_walk != 0;
        auto pace = [&]() {
            if (walk) xcd.pace(1);
        };
        if (ok)
            search_tile<KM, PB, FMT, (FMT != KB_F32)>(
                pace, lds, 0, 1, kChunk, jb.planes, jb.inv_scale, jb.n_img, jb.h, jb.w, jb.disp,
                jb.disp_stride, jb.vel_index, jb.n_vel, reach, k_cand, row, seg, jb.cand_nu,
                jb.cand_alpha, jb.cand_vel, jb.cand_nobs);
        // Generation boundary (as in the single-stack persistent search).
        if (gen < paced) xcd.pace(ok || !walk ? 1 : 1 + paces_inside(jb.n_vel));
    }
}

}  // namespace
}  // namespace kbmi

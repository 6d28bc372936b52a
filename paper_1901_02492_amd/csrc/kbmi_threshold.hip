// Threshold mode and duplicate clustering of libkbmi.
//
//   search_threshold_kernel  every trajectory whose nu reaches a threshold
//                            (Sec. 2.2; Sec. 3.2 keeps nu >= 10), appended
//                            to a device list by wave-wide compaction
//   cluster kernels          groups of hits within eps in (x, y, s*vx, s*vy)
//                            (DBSCAN with min_samples = 1, Sec. 3.3) by
//                            lock-free union-find, and each group's best hit
//
// The threshold search runs the top-k search's own gathers (visit_velocities:
// same table, loads, image order) and score functions, so a hit's nu, alpha
// and n_obs are bitwise the values the top-k path gives that trajectory.  It
// keeps no list, so it needs few registers; it runs in the top-k search's
// paced persistent order with two batches' gathers in flight.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "kbmi_common.h"
#include "kbmi_device.h"

namespace kbmi {
namespace {

constexpr int TH_NV = 16;          // loads of a batch
constexpr int TH_STRIP = 4;        // tiles per strip of the tile order

// One tile: 64 adjacent start pixels of one row, every velocity, with the
// top-k search's gathers (visit_velocities); each trajectory is scored and
// appended if nu >= nu_min: one atomic per wave reserves the wave's slots.
template <class Pace>
__device__ __forceinline__ void threshold_tile(
    Pace &&pace, uint32_t *lds, const float2 *__restrict__ planes, int n_img, int h, int w,
    const GatherEntry *__restrict__ disp, int disp_stride, const int32_t *__restrict__ vel_index,
    int n_vel, int row, int seg, float nu_min, kb_hit *__restrict__ hits, uint64_t cap,
    unsigned long long *__restrict__ n_hits) {
    const int lane = (int)threadIdx.x;
    const int x0 = seg * 64 + lane;
    const uint64_t below = (uint64_t(1) << lane) - 1;
    auto finish = [&](int j, float P, float F, uint32_t c) {
        const float r = inv_sqrt_phi(F);
        const float nu = score_nu(P, F, r);
        const bool pass = x0 < w && nu >= nu_min;
        const uint64_t bal = __ballot(pass);
        if (bal != 0) {
            unsigned long long base = 0;
            if (lane == 0) base = atomicAdd(n_hits, (unsigned long long)__popcll(bal));
            const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base);
            const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
            const uint64_t idx = (((uint64_t)hi << 32) | lo) + (uint64_t)__popcll(bal & below);
            if (pass && idx < cap) {
                kb_hit hit;
                hit.x = x0;
                hit.y = row;
                hit.vel = j;
                hit.nu = nu;
                hit.alpha = score_alpha(P, nu, F, r);
                hit.nobs = (int16_t)c;
                hit.reserved = 0;
                hits[idx] = hit;
            }
        }
    };
    // (Without runs: they gain 4 to 9 % up to 8 images, but with more of them tiles
    // inside run ahead of their XCD's others, 15 x 4096^2, 240 velocities 31.3 -> 35.1 ms.)
    visit_velocities<KB_F32, TH_NV, false>(lds, planes, nullptr, n_img, h, w, disp, disp_stride,
                                           vel_index, n_vel, Reach{}, row, seg, 0, 1, kChunk,
                                           finish, []() { return false; }, []() {}, pace);
}

// Strip tile order, one wave per tile.
__global__ __launch_bounds__(64) void search_threshold_kernel(
    const float2 *__restrict__ planes, int n_img, int h, int w,
    const GatherEntry *__restrict__ disp, int disp_stride, const int32_t *__restrict__ vel_index,
    int n_vel, int nseg, int ntiles, float nu_min, kb_hit *__restrict__ hits, uint64_t cap,
    unsigned long long *__restrict__ n_hits) {
    __shared__ uint32_t lds[kVisitWords];
    int row, seg;
    strip_tile(xcd_remap((int)blockIdx.x, ntiles), nseg, h, TH_STRIP, row, seg);
    threshold_tile([]() {}, lds, planes, n_img, h, w, disp, disp_stride, vel_index, n_vel, row,
                   seg, nu_min, hits, cap, n_hits);
}

// The paced persistent order of the float32 top-k search: per generation each
// XCD covers one block of start pixels and its waves wait (a bounded time) for
// each other at the end of the generation, and inside the tiles of a long walk,
// so that their gathers share the XCD's L2 (25 x 4096^2, 4000 velocities: 1205 ms with
// the generation's pace alone, 685 with both, 1160 before the classes).  The wait
// only shapes timing.
template <bool LONG>
__global__ __launch_bounds__(64) void search_threshold_persistent_kernel(
    const float2 *__restrict__ planes, int n_img, int h, int w,
    const GatherEntry *__restrict__ disp, int disp_stride, const int32_t *__restrict__ vel_index,
    int n_vel, PersistMap pm, float nu_min, kb_hit *__restrict__ hits, uint64_t cap,
    unsigned long long *__restrict__ n_hits, uint32_t *sync) {
    __shared__ uint32_t lds[kVisitWords];
    XcdPace xcd(sync, pm.spin);
    auto pace = [&]() {
        if constexpr (LONG) xcd.pace(1);
    };
    for (int gen = 0; gen < pm.generations; ++gen) {
        int row, seg;
        const bool ok = pm.map(gen, (int)blockIdx.x, row, seg);
        if (ok)
            threshold_tile(pace, lds, planes, n_img, h, w, disp, disp_stride, vel_index, n_vel,
                           row, seg, nu_min, hits, cap, n_hits);
        // Generation boundary.
        xcd.pace(ok || !LONG ? 1 : 1 + paces_inside(n_vel));
    }
}

int threshold_grid() {
    static int cached[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if (cached[dev] == 0) {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &per_cu, search_threshold_persistent_kernel<false>, 64, 0) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 0;
        // (12 and 16 workgroups a CU, which the registers allow, take 19.9 and 19.7 ms
        // for 19.2 at 15 x 2048^2: each XCD's block outgrows its L2.)
        cached[dev] = std::min(per_cu, KBMI_PERSIST_PER_CU) * cus;
    }
    return cached[dev];
}

__global__ void zero_u64_kernel(unsigned long long *p) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0ull;
}

// ---------------------------------------------------------------------------
// Clustering.  parent[] forms a forest in which every edge points to a
// smaller index: uniting two roots hooks the larger under the smaller with a
// compare-and-swap, and a failed swap means the root was hooked meanwhile, to
// a smaller index, so the loop makes progress and ends.  The root of each tree
// is therefore the smallest index of its component.
// ---------------------------------------------------------------------------
constexpr int CL_THREADS = 256;

__device__ inline int cl_load(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline int cl_find(int32_t *parent, int a) {
    int p = cl_load(parent + a);
    while (p != a) {
        a = p;
        p = cl_load(parent + a);
    }
    return a;
}

__device__ inline void cl_unite(int32_t *parent, int a, int b) {
    for (;;) {
        a = cl_find(parent, a);
        b = cl_find(parent, b);
        if (a == b) return;
        if (a > b) {
            const int t = a;
            a = b;
            b = t;
        }
        const int old = atomicCAS(parent + b, b, a);
        if (old == b) return;
        b = old;
    }
}

// Pairs are found through a grid of cells of side c = eps (1 + 2^-20) over
// the four coordinates (x, y, u, v), u = s * vx, v = s * vy: two hits within
// distance eps differ by at most eps in every coordinate, so their cells
// differ by at most one in every coordinate, and each hit only meets the hits
// of its own and the 80 neighbouring cells.  The cells sit in an
// open-addressing hash table (cell key -> list of the cell's hits).  Pair
// (i, j) is joined when d2 <= eps2 with
// d2 = ((dx*dx + dy*dy) + du*du) + dv*dv in double.  A hit whose velocity
// index is outside the grid gets no cell: it stays a group of its own.
//
// Being neighbours is symmetric, so a hit looks for the 40 neighbours on one
// side only (offsets that are positive in their last nonzero coordinate) and
// is found by the hits of the other 40; its own cell is the rest of the list
// it was pushed onto.  Most of the 40 are empty, and the table (12 bytes a
// slot, 100 MB for 4e6 hits) is in no cache, so a bitmap of the occupied
// cells is asked first: bit (a & 63) of word hash(a >> 6, b, c, d), four bits
// per table slot (4 MB for 4e6 hits, an XCD's L2), so that the three cells of
// a neighbouring (b, c, d) are nearly always one word: 14 words, all in
// flight together, stand for 81 probes in series, and the table is probed
// for set bits alone.  A call on 4e6 hits: 6.76 -> 1.84 ms,
// 1.67 with neighbours' keys by constants and set bits read, not set again.
__device__ inline double2 cl_vel(const double2 *vel, int n_vel, int j) {
    return (unsigned)j < (unsigned)n_vel ? vel[j] : make_double2(NAN, NAN);
}

constexpr uint64_t kEmptyCell = ~0ull;

__device__ inline int64_t cl_cell(double coord, double inv_c) {
#pragma clang fp contract(off)
    const double q = floor(coord * inv_c);
    return (int64_t)fmin(fmax(q, -4.0e18), 4.0e18);
}

// 64-bit key of cell (a, b, c, d): a finalising mix of a packed sum (distinct
// cells may share a key, which only adds hits whose distance is then tested).
// A neighbour's sum differs by constants, so it takes no products of its own
// (64-bit products are what a key costs: four in the sum, two in the mix).
constexpr uint64_t kClA = 0x9E3779B97F4A7C15ull, kClB = 0xC2B2AE3D27D4EB4Full,
                   kClC = 0x165667B19E3779F9ull, kClD = 0xD6E8FEB86659FD93ull;
__device__ inline uint64_t cl_sum(int64_t a, int64_t b, int64_t c, int64_t d) {
    return (uint64_t)a * kClA + (uint64_t)b * kClB + (uint64_t)c * kClC + (uint64_t)d * kClD;
}
__device__ inline uint64_t cl_key_of(uint64_t z) {
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z == kEmptyCell ? kEmptyCell - 1 : z;
}
// step - 1 of one coordinate, step in 0 .. 2.
__device__ inline uint64_t cl_step(int step, uint64_t k) {
    return step == 0 ? 0 - k : step == 2 ? k : 0;
}
// The sum's change for group o of the cells around one: (b, c, d) = offset + 1
// in base 3.
__device__ inline uint64_t cl_group(int o) {
    return cl_step(o % 3, kClB) + cl_step(o / 3 % 3, kClC) + cl_step(o / 9, kClD);
}

struct ClHit {
    double x, y, u, v;
    bool ok;
};

__device__ inline ClHit cl_hit(const kb_hit *hits, const double2 *vel, int n_vel, double s,
                               int i) {
#pragma clang fp contract(off)
    const kb_hit h = hits[i];
    const double2 vj = cl_vel(vel, n_vel, h.vel);
    ClHit r;
    r.x = (double)h.x;
    r.y = (double)h.y;
    r.u = s * vj.x;
    r.v = s * vj.y;
    r.ok = (unsigned)h.vel < (unsigned)n_vel;
    return r;
}

// Bitmap words per table slot: 1 / 16 (four bits a slot).
constexpr int CL_SLOTS_PER_WORD = 16;

__global__ void cl_init_kernel(int32_t *parent, int n, uint64_t *table_key, int32_t *table_head,
                               uint64_t *bitmap, int64_t slots) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < slots;
         i += (int64_t)gridDim.x * blockDim.x) {
        table_key[i] = kEmptyCell;
        table_head[i] = -1;
        if (i < n) parent[i] = (int32_t)i;
        if (i < slots / CL_SLOTS_PER_WORD) bitmap[i] = 0;
    }
}

// Hit i joins the list of its cell (pushed at the head; the lists are read by
// the next kernel only).
__global__ __launch_bounds__(CL_THREADS) void cl_insert_kernel(
    const kb_hit *__restrict__ hits, int n, const double2 *__restrict__ vel, int n_vel, double s,
    double inv_c, uint64_t *table_key, int32_t *table_head, uint64_t mask, uint64_t *bitmap,
    int32_t *__restrict__ next) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= n) return;
    const ClHit h = cl_hit(hits, vel, n_vel, s, i);
    next[i] = -1;
    if (!h.ok) return;
    const int64_t a = cl_cell(h.x, inv_c), b = cl_cell(h.y, inv_c), c = cl_cell(h.u, inv_c),
                  d = cl_cell(h.v, inv_c);
    // Hits of one cell come in numbers: what an earlier one has set is read
    // instead of set again (an atomic is the dearer access).
    uint64_t *word = bitmap + (cl_key_of(cl_sum(a >> 6, b, c, d)) & (mask / CL_SLOTS_PER_WORD));
    const uint64_t bit = 1ull << (a & 63);
    if (!(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit))
        atomicOr(reinterpret_cast<unsigned long long *>(word), bit);
    const uint64_t key = cl_key_of(cl_sum(a, b, c, d));
    uint64_t slot = key & mask;
    for (;;) {
        uint64_t prev =
            __hip_atomic_load(table_key + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == kEmptyCell)
            prev = atomicCAS(reinterpret_cast<unsigned long long *>(table_key + slot),
                             (unsigned long long)kEmptyCell, (unsigned long long)key);
        if (prev == kEmptyCell || prev == key) {
            next[i] = atomicExch(table_head + slot, i);
            return;
        }
        slot = (slot + 1) & mask;   // the table has at least twice as many slots as hits
    }
}

__global__ __launch_bounds__(CL_THREADS) void cl_grid_pairs_kernel(
    const kb_hit *__restrict__ hits, int n, const double2 *__restrict__ vel, int n_vel, double s,
    double inv_c, double eps2, const uint64_t *__restrict__ table_key,
    const int32_t *__restrict__ table_head, uint64_t mask, const uint64_t *__restrict__ bitmap,
    const int32_t *__restrict__ next, int32_t *parent) {
#pragma clang fp contract(off)
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= n) return;
    const ClHit hi = cl_hit(hits, vel, n_vel, s, i);
    if (!hi.ok) return;
    const int64_t c0 = cl_cell(hi.x, inv_c), c1 = cl_cell(hi.y, inv_c);
    const int64_t c2 = cl_cell(hi.u, inv_c), c3 = cl_cell(hi.v, inv_c);
    const uint64_t word_mask = mask / CL_SLOTS_PER_WORD;
    // Joins the hits of a list from hit j on that are within eps.
    auto join = [&](int j) {
        for (; j >= 0; j = next[j]) {
            const ClHit hj = cl_hit(hits, vel, n_vel, s, j);
            const double dx = hi.x - hj.x, dy = hi.y - hj.y, du = hi.u - hj.u, dv = hi.v - hj.v;
            const double dd = ((dx * dx + dy * dy) + du * du) + dv * dv;
            if (dd <= eps2) cl_unite(parent, i, j);
        }
    };
    join(next[i]);
    // The words of the 14 groups of three cells a - 1, a, a + 1; the groups
    // are numbered (b, c, d) = offset + 1 in base 3, the hit's own is 13.
    const int bit = (int)(c0 & 63);
    const bool edge = bit == 0 || bit == 63;
    const uint64_t words = cl_sum(c0 >> 6, c1, c2, c3);
    uint64_t word[14];
#pragma unroll
    for (int g = 0; g < 14; ++g) word[g] = bitmap[cl_key_of(words + cl_group(g + 13)) & word_mask];
    // Bit 3 g + e of `probe`: cell a + e - 1 of group g may hold hits.
    uint64_t probe = 0;
#pragma unroll
    for (int g = 0; g < 14; ++g)
        probe |= (bit > 0 ? (word[g] >> (bit - 1)) & 7u : (word[g] << 1) & 7u) << (3 * g);
    if (edge) {   // the third cell is in the word beside
        const uint64_t beside = words + (bit == 0 ? 0 - kClA : kClA);
        const int e = bit == 0 ? 0 : 2;
#pragma unroll
        for (int g = 0; g < 14; ++g) {
            const uint64_t wd = bitmap[cl_key_of(beside + cl_group(g + 13)) & word_mask];
            probe |= ((wd >> (bit == 0 ? 63 : 0)) & 1u) << (3 * g + e);
        }
    }
    probe &= ~uint64_t(3);   // a - 1 and a of the hit's own group
    const uint64_t cell = cl_sum(c0, c1, c2, c3);
    while (probe != 0) {
        const int p = __builtin_ctzll(probe);
        probe &= probe - 1;
        const uint64_t key = cl_key_of(cell + cl_step(p % 3, kClA) + cl_group(p / 3 + 13));
        uint64_t slot = key & mask;
        for (;;) {
            const uint64_t k = table_key[slot];
            if (k == kEmptyCell) break;
            if (k == key) {
                join(table_head[slot]);
                break;
            }
            slot = (slot + 1) & mask;
        }
    }
}

// The roots, and the empty state of each group's best hit.
__global__ void cl_flatten_kernel(int32_t *parent, uint32_t *best_nu, uint64_t *best_key,
                                  int32_t *rep_of_root, int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) {
        parent[i] = cl_find(parent, i);
        best_nu[i] = 0u;
        best_key[i] = ~0ull;
        rep_of_root[i] = -1;
    }
}

__device__ inline uint64_t cl_key(const kb_hit &h) {
    return ((uint64_t)(uint32_t)h.y << 40) | ((uint64_t)(uint32_t)h.x << 16) |
           (uint64_t)(uint32_t)h.vel;
}

__global__ void cl_best_nu_kernel(const kb_hit *__restrict__ hits, const int32_t *root,
                                  uint32_t *best_nu, int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) atomicMax(best_nu + root[i], nu_order_bits(hits[i].nu));
}

__global__ void cl_best_key_kernel(const kb_hit *__restrict__ hits, const int32_t *root,
                                   const uint32_t *best_nu, uint64_t *best_key, int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) {
        const kb_hit h = hits[i];
        const int r = root[i];
        if (nu_order_bits(h.nu) == best_nu[r])
            atomicMin(reinterpret_cast<unsigned long long *>(best_key + r),
                      (unsigned long long)cl_key(h));
    }
}

__global__ void cl_rep_kernel(const kb_hit *__restrict__ hits, const int32_t *root,
                              const uint32_t *best_nu, const uint64_t *best_key,
                              int32_t *rep_of_root, int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) {
        const kb_hit h = hits[i];
        const int r = root[i];
        if (nu_order_bits(h.nu) == best_nu[r] && cl_key(h) == best_key[r]) rep_of_root[r] = i;
    }
}

__global__ void cl_out_kernel(const int32_t *root, const int32_t *rep_of_root, int32_t *rep,
                              int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) rep[i] = rep_of_root[root[i]];
}

size_t r256(size_t n) { return (n + 255) & ~static_cast<size_t>(255); }

struct ClusterLayout {
    size_t parent, best_nu, best_key, rep_of_root, vel, next, table_key, table_head, total;
    uint64_t slots;   // hash-table slots: a power of two >= 2 * n_hits
};

ClusterLayout cluster_layout(int64_t n_hits, int64_t n_vel) {
    ClusterLayout l{};
    const size_t n = static_cast<size_t>(n_hits);
    l.slots = 64;
    while (l.slots < 2 * static_cast<uint64_t>(n)) l.slots <<= 1;
    l.parent = 0;
    l.best_nu = l.parent + r256(n * sizeof(int32_t));
    l.best_key = l.best_nu + r256(n * sizeof(uint32_t));
    // (best_key's space holds the bitmap first.)
    l.rep_of_root = l.best_key + r256(std::max<uint64_t>(n * sizeof(uint64_t),
                                                         l.slots / CL_SLOTS_PER_WORD * 8));
    l.vel = l.rep_of_root + r256(n * sizeof(int32_t));
    l.next = l.vel + r256(static_cast<size_t>(n_vel) * 2 * sizeof(double));
    l.table_key = l.next + r256(n * sizeof(int32_t));
    l.table_head = l.table_key + r256(l.slots * sizeof(uint64_t));
    l.total = l.table_head + r256(l.slots * sizeof(int32_t));
    return l;
}

kb_status launch_threshold(const float *psi_phi, int64_t n_img, int64_t h, int64_t w,
                           int64_t n_vel, float nu_min, kb_hit *hits, int64_t max_hits,
                           uint64_t *n_hits, void *workspace, hipStream_t s) {
    char *ws = static_cast<char *>(workspace);
    const WorkspaceLayout lay = workspace_layout(n_img, h, w, n_vel);
    const int nseg = (int)((w + 63) / 64);
    const int64_t ntiles = (int64_t)nseg * h;
    const int grid = threshold_grid();
    const int per_xcd = grid / 8;
    const GatherEntry *disp = reinterpret_cast<const GatherEntry *>(ws + lay.table);
    const int32_t *order = reinterpret_cast<const int32_t *>(ws + lay.order);
    if (grid >= 8 && grid % 8 == 0 && per_xcd % KBMI_PERSIST_BS == 0 &&
        ntiles >= 4 * (int64_t)grid) {
        PersistMap pm;
        pm.nseg = nseg;
        pm.h = (int)h;
        pm.bs = KBMI_PERSIST_BS;
        pm.brows = per_xcd / KBMI_PERSIST_BS;
        pm.nbc = (nseg + pm.bs - 1) / pm.bs;
        pm.nbr = ((int)h + pm.brows - 1) / pm.brows;
        pm.generations = block_generations(pm.nbc, pm.nbr);
        pm.spin = KBMI_PERSIST_SPIN;
        pm.long_walk = is_long_walk(n_img, n_vel, true);
        uint32_t *sync = reinterpret_cast<uint32_t *>(ws + lay.sync);
        hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(64), 0, s, sync, 8);
        kb_status st = launch_status("zero_words_kernel");
        if (st != KB_OK) return st;
        hipLaunchKernelGGL((pm.long_walk ? search_threshold_persistent_kernel<true>
                                         : search_threshold_persistent_kernel<false>),
                           dim3((unsigned)grid), dim3(64), 0, s,
                           reinterpret_cast<const float2 *>(psi_phi), (int)n_img, (int)h, (int)w,
                           disp, (int)table_stride(n_img), order, (int)n_vel, pm, nu_min, hits,
                           (uint64_t)max_hits, reinterpret_cast<unsigned long long *>(n_hits),
                           sync);
        return launch_status("search_threshold_persistent_kernel");
    }
    hipLaunchKernelGGL(search_threshold_kernel, dim3((unsigned)ntiles), dim3(64), 0, s,
                       reinterpret_cast<const float2 *>(psi_phi), (int)n_img, (int)h, (int)w,
                       disp, (int)table_stride(n_img), order, (int)n_vel, nseg, (int)ntiles,
                       nu_min, hits, (uint64_t)max_hits,
                       reinterpret_cast<unsigned long long *>(n_hits));
    return launch_status("search_threshold_kernel");
}

}  // namespace
}  // namespace kbmi

using namespace kbmi;

extern "C" {

kb_status kb_search_threshold(const float *psi_phi, int64_t n_img, int64_t h, int64_t w,
                              const double *t, const double *vel, int64_t n_vel, float nu_min,
                              kb_hit *hits, int64_t max_hits, uint64_t *n_hits, void *workspace,
                              size_t workspace_bytes, void *stream) {
    clear_error();
    if (!psi_phi || !t || !vel || !n_hits || (!hits && max_hits > 0))
        return fail(KB_EINVAL, "planes, times, velocities, the hit list and its counter must "
                               "be non-null");
    kb_status st = check_frame(n_img, h, w);
    if (st != KB_OK) return st;
    if (n_vel < 1 || n_vel > 65535)
        return fail(KB_EINVAL, "n_vel must be in [1, 65535] (got %lld)", (long long)n_vel);
    if (max_hits < 0) return fail(KB_EINVAL, "max_hits must be >= 0");
    if (!std::isfinite(nu_min)) return fail(KB_EINVAL, "nu_min must be finite");
    if (w >= (int64_t(1) << 24) || h >= (int64_t(1) << 24))
        return fail(KB_EUNSUPPORTED, "threshold mode takes frames below 2^24 on each side");
    st = check_times_velocities(t, n_img, vel, n_vel);
    if (st != KB_OK) return st;
    if (!workspace) return fail(KB_EINVAL, "the threshold search needs a workspace");
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
        return fail(KB_EINVAL, "workspace must be 256-byte aligned");
    const WorkspaceLayout lay = workspace_layout(n_img, h, w, n_vel);
    if (workspace_bytes < lay.total)
        return fail(KB_ENOMEM, "workspace needs %zu bytes (got %zu)", lay.total, workspace_bytes);
    hipStream_t s = (hipStream_t)stream;
    st = upload_table(t, n_img, vel, n_vel, h, w, 8, workspace, s);
    if (st != KB_OK) return st;
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(64), 0, s,
                       reinterpret_cast<unsigned long long *>(n_hits));
    st = launch_status("zero_u64_kernel");
    if (st != KB_OK) return st;
    return launch_threshold(psi_phi, n_img, h, w, n_vel, nu_min, hits, max_hits, n_hits,
                            workspace, s);
}

size_t kb_cluster_workspace_bytes(int64_t n_hits, int64_t n_vel) {
    if (n_hits < 0 || n_vel < 1) return 0;
    return cluster_layout(n_hits, n_vel).total;
}

kb_status kb_cluster_hits(const kb_hit *hits, int64_t n_hits, const double *vel, int64_t n_vel,
                          double s, double eps, int32_t *rep, void *workspace,
                          size_t workspace_bytes, void *stream) {
    clear_error();
    if (n_hits < 0) return fail(KB_EINVAL, "n_hits must be >= 0");
    if (n_hits == 0) return KB_OK;
    if (!hits || !vel || !rep || !workspace)
        return fail(KB_EINVAL, "hits, velocities, rep and workspace must be non-null");
    if (n_vel < 1 || n_vel > 65535)
        return fail(KB_EINVAL, "n_vel must be in [1, 65535] (got %lld)", (long long)n_vel);
    if (n_hits > (int64_t(1) << 30))
        return fail(KB_EUNSUPPORTED, "at most 2^30 hits per call");
    if (!(std::isfinite(s) && s >= 0.0)) return fail(KB_EINVAL, "s must be finite and >= 0");
    if (!(std::isfinite(eps) && eps >= 0.0)) return fail(KB_EINVAL, "eps must be finite and >= 0");
    for (int64_t j = 0; j < 2 * n_vel; ++j)
        if (!std::isfinite(vel[j])) return fail(KB_EINVAL, "velocities must be finite");
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
        return fail(KB_EINVAL, "workspace must be 256-byte aligned");
    const ClusterLayout lay = cluster_layout(n_hits, n_vel);
    if (workspace_bytes < lay.total)
        return fail(KB_ENOMEM, "workspace needs %zu bytes (got %zu)", lay.total, workspace_bytes);
    hipStream_t st_ = (hipStream_t)stream;
    char *ws = static_cast<char *>(workspace);
    kb_status st = staged_copy(ws + lay.vel, vel, static_cast<size_t>(2 * n_vel) * sizeof(double),
                               st_);
    if (st != KB_OK) return st;
    int32_t *parent = reinterpret_cast<int32_t *>(ws + lay.parent);
    uint32_t *best_nu = reinterpret_cast<uint32_t *>(ws + lay.best_nu);
    uint64_t *best_key = reinterpret_cast<uint64_t *>(ws + lay.best_key);
    int32_t *rep_of_root = reinterpret_cast<int32_t *>(ws + lay.rep_of_root);
    const double2 *dvel = reinterpret_cast<const double2 *>(ws + lay.vel);
    const int n = (int)n_hits;
    const dim3 b1((unsigned)((n + 255) / 256)), t1(256);
    uint64_t *table_key = reinterpret_cast<uint64_t *>(ws + lay.table_key);
    int32_t *table_head = reinterpret_cast<int32_t *>(ws + lay.table_head);
    int32_t *next = reinterpret_cast<int32_t *>(ws + lay.next);
    const uint64_t mask = lay.slots - 1;
    // Cells slightly wider than eps, so that rounding in coordinate / side
    // never separates two hits at distance eps by two cells (eps = 0: cells
    // of side 1; only identical hits join).
    const double side = eps > 0.0 ? eps * (1.0 + 0x1p-20) : 1.0;
    const double inv_c = 1.0 / side;
    // The bitmap lies in best_key's space, which is written after its last use.
    uint64_t *bitmap = best_key;
    hipLaunchKernelGGL(cl_init_kernel,
                       dim3((unsigned)std::min<uint64_t>(2048, (lay.slots + 255) / 256)),
                       dim3(256), 0, st_, parent, n, table_key, table_head, bitmap,
                       (int64_t)lay.slots);
    if ((st = launch_status("cl_init_kernel")) != KB_OK) return st;
    hipLaunchKernelGGL(cl_insert_kernel, b1, dim3(CL_THREADS), 0, st_, hits, n, dvel, (int)n_vel,
                       s, inv_c, table_key, table_head, mask, bitmap, next);
    if ((st = launch_status("cl_insert_kernel")) != KB_OK) return st;
    hipLaunchKernelGGL(cl_grid_pairs_kernel, b1, dim3(CL_THREADS), 0, st_, hits, n, dvel,
                       (int)n_vel, s, inv_c, eps * eps, table_key, table_head, mask, bitmap, next,
                       parent);
    if ((st = launch_status("cl_grid_pairs_kernel")) != KB_OK) return st;
    hipLaunchKernelGGL(cl_flatten_kernel, b1, t1, 0, st_, parent, best_nu, best_key, rep_of_root,
                       n);
    if ((st = launch_status("cl_flatten_kernel")) != KB_OK) return st;
    hipLaunchKernelGGL(cl_best_nu_kernel, b1, t1, 0, st_, hits, parent, best_nu, n);
    if ((st = launch_status("cl_best_nu_kernel")) != KB_OK) return st;
    hipLaunchKernelGGL(cl_best_key_kernel, b1, t1, 0, st_, hits, parent, best_nu, best_key, n);
    if ((st = launch_status("cl_best_key_kernel")) != KB_OK) return st;
    hipLaunchKernelGGL(cl_rep_kernel, b1, t1, 0, st_, hits, parent, best_nu, best_key,
                       rep_of_root, n);
    if ((st = launch_status("cl_rep_kernel")) != KB_OK) return st;
    hipLaunchKernelGGL(cl_out_kernel, b1, t1, 0, st_, parent, rep_of_root, rep, n);
    return launch_status("cl_out_kernel");
}

}  // extern "C"

// te_internal.h -- structures shared by the host runtime and the HIP kernels of libte.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

namespace te {

// Largest supported embedding dimensions and neighbour count.
constexpr int kMaxDimY = 4;
constexpr int kMaxDimX = 4;
constexpr int kMaxK = 15;
constexpr int kWave = 64;                 // wavefront width on gfx950
constexpr int kMaxWavesPerWG = 4;         // search kernel workgroup: up to 4 independent waves

// One search space ("chunk", eq. 10 pooled points) as the kernels see it.
// Coordinate m of point j lives at
//   base[tp + m * ld + j]                 for m <  1 + d_y  (y_t' and target past)
//   base[s + (m - 1 - d_y) * ld + j]      for m >= 1 + d_y  (source past)
// so the originals and surrogates of one window share the (y_t', Y_past) block.
// In an ordered chunk ld is n, and base[geo + (2 m) nb + b], base[geo + (2 m + 1) nb + b]
// are the smallest and largest target-past coordinate m < d_y of points 64 b .. 64 b + 63
// (nb = ceil(n / 64); a chunk of one block has none).
struct ChunkDesc {
    int64_t tp;       // float offset of the target block
    int64_t s;        // float offset of the source block
    int64_t geo;      // ordered chunks: float offset of the block boxes; else: ld, the stride between coordinates
    int64_t out;      // per-point output offset (eps / counts), or -1
    int64_t pbase;    // index in the partial-sum array of the chunk's block 0
    int64_t perm;     // offset in perm_base of the sorted-to-original point map, or -1
    int32_t n;        // points in the chunk
    int32_t item0;    // launch work-item index of the first scheduled block
    int32_t block0;   // first scheduled block (64 references) of the chunk
    int32_t result;   // slot of the chunk's estimate in the result array
};

// Work for the embedding kernel: writes one chunk's source block, and the
// target block when tp >= 0.
struct EmbedTask {
    int64_t tp;       // float offset of the target block, or -1
    int64_t s;        // float offset of the source block
    int64_t perm;     // int32 offset of the source permutation row in the batch's permutation area, or -1 (identity)
    int64_t sig;      // int32 offset of the window's sorted-to-original point map, or -1 (identity)
    int32_t pair, w, W, Rc;
    int32_t n;        // Rc * W
    int32_t u;        // source delay of this block; 0: the launch's delay
    int32_t u_slot;   // > 0: the delay is read on the device from u_dev[u_slot - 1] (overrides u)
    int32_t box;      // writes the block boxes: -1 no, 0 behind the order map, > 0 in the key scratch at
                      // (box - 1) * kBoxScratchUnit
};

// One surrogate's trial permutation in a batch's permutation area.  It is either
// copied from the caller's [pair][point][surrogate][trial] array (and checked to
// be a permutation of 0..rc-1) or drawn on the device from the problem's seed,
// keyed by (pair, point, surr).  Entries rc..len-1 of a written row are the
// identity.
struct PermTask {
    int64_t src;      // int32 offset of the row in the caller's array (copy mode)
    int64_t dst;      // int32 offset of the row in the destination
    int32_t rc;       // trials pooled by the window: the row permutes 0..rc-1
    int32_t len;      // entries written (>= rc)
    int32_t pair, point, surr, pad_;
};

// Ordering of one search space: 64 consecutive points of the order (a block) are
// close together in the target past (order_kernel).  The map's entry q, at sigma + sig
// (order_at in te_device.h), is the original index of the point at position q.
struct SortTask {
    int64_t sig;      // int32 offset of the output map
    int64_t scratch;  // uint64 offset of global key scratch (npad > kSortLds), else -1
    int64_t key_off;  // mode 1: float offset of the first target-past coordinate (point q at key_off + q)
    int32_t mode;     // 0: keys from y of window point q = r W + (t' - w); 1: stored coordinates
    int32_t pair, w, W, Rc, n, npad;
    int32_t nd;       // coordinates that order the space; 0: the launch's d_y
};
constexpr int kSortLds = 16384;   // keys sorted in LDS (128 KiB) up to this many (padded) points

// Where the block boxes of an ordered space of n points live: up to kSortLds points in the
// words behind its 16-bit map, above that in its key scratch, which the ordering is done with.
constexpr int64_t box_words_behind_map(int64_t n) { return (n + 1) / 2; }
constexpr int kBoxScratchUnit = 2 * kSortLds;   // scratch offsets are multiples of this many keys

// Slabs: runs of whole blocks.  A run of `leaves` blocks is cut along one coordinate into as many
// slabs as the rem-th root of their number, rounded, when rem coordinates (this one included) are
// left, so that every coordinate gets its share; slab i of s holds blocks [slab_first(i), slab_first(i + 1)).
__host__ __device__ constexpr int slab_count(int leaves, int rem)
{
    if (rem <= 1)
        return 1;
    int s = 1;
    for (;; ++s) {
        int64_t p = 1;                    // (s + 1/2)^rem against leaves, both times 2^rem
        for (int j = 0; j < rem; ++j)
            p *= 2 * s + 1;
        if (p > ((int64_t)leaves << rem))
            return s;
    }
}
__host__ __device__ constexpr int slab_first(int leaves, int slabs, int i) { return (int)((int64_t)leaves * i / slabs); }

// A space of more than kSlabMax points is first cut into slabs of at most that many, which
// workgroups of their own then order in LDS.  Up to kMaxSlabs x kSlabMax points split_kernel cuts
// it, above that a sort by the first coordinate (whole_tiles_kernel).
constexpr int kSlabMax = 8192;
constexpr int kMaxSlabs = 64;
__host__ __device__ constexpr bool sorted_whole(int n) { return n > kMaxSlabs * kSlabMax; }
__host__ __device__ constexpr int order_slabs(int n, int nd)
{
    if (n <= kSlabMax)
        return 1;
    const int nl = (n - 1) / kWave + 1;
    const int least = (nl + kSlabMax / kWave - 1) / (kSlabMax / kWave);   // slabs of at most kSlabMax points
    int s = slab_count(nl, nd);
    s = s < least ? least : s;
    return s > kMaxSlabs && !sorted_whole(n) ? kMaxSlabs : s;
}

// What the launches that order a table of tasks, longest first, need to know of it.
struct SortSizes {
    int n_tasks = 0;
    int max_n = 0;    // points of the longest
    int n_cut = 0;    // tasks above kSlabMax points
    int n_whole = 0;  // tasks that are sorted whole
    void add(int n)
    {
        ++n_tasks;
        max_n = max_n < n ? n : max_n;
        n_cut += n > kSlabMax;
        n_whole += sorted_whole(n);
    }
};

// Copy of one pre-embedded chunk into its order, with its block boxes:
// dst[dst + m n + q] = src[src + m ld + map[q]].
struct GatherTask {
    int64_t src, ld, dst, sig;
    int32_t n;
    int32_t box;      // boxes in the key scratch (n > kSortLds): its offset / kBoxScratchUnit
};

// Arguments of the search kernel (passed by value; read from the kernarg segment).
struct SearchArgs {
    const float *base;          // coordinate storage
    const ChunkDesc *chunks;    // [n_chunks] in schedule order
    const int32_t *item_start;  // [n_chunks] chunks[c].item0, ascending
    int32_t n_chunks;
    int32_t n_items;
    int32_t k;
    int32_t pad_;
    int32_t *counter;           // work-queue head, zero before launch
    double *partial;            // [n_items] per-item sum of psi terms
    float *eps_out;             // optional per-point radius
    int32_t *cnt_out;           // optional per-point counts [3][cnt_stride]
    int64_t cnt_stride;
    const int32_t *perm_base;   // sorted-to-original point maps (per-point outputs only)
    unsigned long long *work;   // optional: [0] += pairs evaluated in pass 1, [1] += in pass 2 (a pair per chunk),
                                // [2], [3] += the same counted once per set of chunks
    double *lte_out;            // optional per-point local TE (at out + original index)
    int32_t sorted;             // chunks are in order_kernel's order, with block boxes
    int32_t n_parts;            // > 1: items split into n_parts queues (counter[p] heads queue p), see kQueues
    const int32_t *part_start;  // [n_parts + 1] first item of each queue (n_parts > 1)
    const int32_t *set_first;   // non-null: chunk-set search; n_chunks counts sets, set c holds the chunks
                                // [set_first[c], set_first[c+1]) (at most set_variants(d_y, d_x)), item_start is per set
};

// Chunks of one window searched together by the chunk-set search (they share the
// (y_t', Y_past) block and its order and differ in the source block).  More of them share a pair's
// target differences, but a block of candidates has to be examined for the chunk with the largest
// radius.  Measured, us, two / three / four to a set (8 windows of 20 000 points x 61 chunks):
// (1, 3) 19 939 / 20 189 / 23 806, (2, 2) 7 978 / 7 601 / 8 073, (3, 3) 12 530 / 12 873 / 13 109,
// (4, 4) 19 773 / 19 796 / -; 40 windows of 2 400 points x 101: (3, 3) 4 704 / 4 434 / 4 386,
// (4, 4) 5 995 / 5 738 / 6 247; with one source coordinate: (1, 1) 2 592 / 2 497 / 2 367,
// (2, 1) 2 738 / 2 573 / 2 399.  Two are 1 to 3 % ahead on large windows at (1, 3) and (3, 3) and 4 to 6 %
// behind on small ones, so three serve all sizes.
constexpr int set_variants(int d_y, int d_x)
{
    return d_x == 1 ? 4 : 3;
}
constexpr int kMaxSetVariants = 4;

// Points per window (pooled chunk) at most: the set search addresses coordinate m of a
// block as a 32-bit byte offset 4 (m ld + j) from the block's start, m <= 4 and ld = N.
constexpr int kMaxWindowPoints = 1 << 27;

// Work queues of a batched search: one per XCD of an MI355X.  Workgroups are
// dispatched to the XCDs round-robin, so the waves of workgroup g start on queue
// g % kQueues and a chunk's coordinates stay in one XCD's L2; a wave whose queue
// is empty moves on to the next one.
constexpr int kQueues = 8;

// Tunable launch shape of the search kernel.
struct SearchConfig {
    int slots;        // candidate blocks counted together in pass 2: 4 -> one, 8 and 16 -> two
    int waves_per_wg; // independent wavefronts per workgroup
    int wg_per_cu;    // persistent workgroups per compute unit
    bool timed = false;   // the tuners: persistent waves however small the launch is, so that a shape is what is timed
};

struct DeviceInfo {
    int device = -1;
    int n_cu = 0;
    char arch[64] = {0};
};

// Kernel launchers (te_kernels.hip).  All return hipSuccess or the launch error.
hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t st);
hipError_t launch_embed(const float *x, const float *y, const int32_t *perms, int32_t *sigma, uint64_t *scratch,
                        const int32_t *u_dev, const EmbedTask *tasks, int n_tasks, int max_n, float *base, int R,
                        int T, int d_y, int d_x, int tau, int u, int cond, int32_t *err, hipStream_t st);
// Order maps of the tasks' search spaces (longest first) by their d_y target-past coordinates (0: the
// tasks' own, at most 4; ld: the stride between the coordinates of pts, mode 1; tau: the embedding
// delay, mode 0).
hipError_t launch_sort(const float *y, const float *pts, int64_t ld, const SortTask *tasks, const SortSizes &sizes,
                       int32_t *sigma, uint64_t *scratch, int R, int T, int d_y, int tau, hipStream_t st);
hipError_t launch_gather(const float *src, const GatherTask *tasks, int n_tasks, int max_n, int32_t *sigma,
                         uint64_t *scratch, float *dst, int D, int d_y, hipStream_t st);
// Fill a batch's permutation area: copy (and check) the caller's rows when src is
// given, else draw every row (of at most max_rc trials) from `seed`.  Sets bit 2 of *err for an invalid row.
hipError_t launch_perms(const int32_t *src, const PermTask *tasks, int n_tasks, int max_rc, int32_t *dst,
                        uint64_t seed, int32_t *err, hipStream_t st);
hipError_t launch_search(const SearchArgs &a, int d_y, int d_x, const SearchConfig &cfg, int grid_waves,
                         hipStream_t st);
// A kernel of the search over ordered chunks and its dynamic LDS bytes (te_search.hip).
struct ordered_search {
    void (*fn)(SearchArgs);
    size_t lds;
};
ordered_search pick_ordered(int d_y, int d_x, int k, int slots, bool sets, int waves_per_wg);
int waves_to_a_block(int64_t n_items, int set_coords, int k, bool queues);
ordered_search pick_shared(int d_y, int d_x, int k, bool sets, int w);
// With pv != nullptr the launch also computes the n_groups p-values (results laid
// out [group][original, surrogates...]; NaN when *err is set) and copies *err to
// *err_out when that is given: in its last-finishing workgroup, counted on `done`
// (zero before the launch), for small grids, else in a second kernel.
hipError_t launch_reduce(const ChunkDesc *chunks, int n_chunks, const double *partial, int k,
                         const int32_t *err, double *results, hipStream_t st, int n_groups = 0, int n_surr = 0,
                         double *pv = nullptr, int32_t *done = nullptr, int32_t *err_out = nullptr);
hipError_t launch_pvalues(const double *results, int n_groups, int n_surr, double *pv, hipStream_t st);
hipError_t launch_argmax_u(const double *results, int n_groups, int n_u, const int32_t *u_values, int32_t *u_sel,
                           hipStream_t st);
bool search_supported(int d_y, int d_x, int k, int slots);
bool search_sets_supported(int d_y, int d_x, int k);
// Resident workgroups per compute unit of the chunk-set search (0 if unknown).
int search_sets_occupancy(int d_y, int d_x, int slots, int waves_per_wg);
unsigned long long *work_counters();   // this device's evaluated-pair counters [4] (measurement)

// Search launch bracketed by profiling events when measurement is enabled (te_profile.cpp).
hipError_t launch_search_timed(const SearchArgs &a, int d_y, int d_x, const SearchConfig &cfg, int grid_waves,
                               hipStream_t st);

}  // namespace te

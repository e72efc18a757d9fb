// te_kernels.hip -- HIP kernels of libte for gfx950 (CDNA4, wave64) around the search.
//
//   split_kernel, whole_*_kernel, order_kernel  order a search space so that
//                    64 consecutive points are close together in the target past.
//   embed_kernel     eq. 6-7 / eq. 10: gathers the pooled points of a window
//                    from the raw [pair][trial][sample] series into
//                    coordinate-major blocks; bit copies only.
//   search_unordered_kernel  the KSG type-1 searches (text before eq. 9) over
//                    chunks in the caller's order; the searches over ordered
//                    chunks are in te_search.hip.
//   reduce_kernel    eq. 9/10 per chunk: psi(k) + mean of the terms.
//   pvalue_kernel    fraction of surrogate estimates >= the original.
//   argmax_u_kernel  eq. 5: the assumed delay with the largest estimate.
//   take_perms_kernel, draw_perms_kernel  the surrogates' trial permutations.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "te_device.h"
#include "te_internal.h"

namespace te {

namespace {

// ------------------------------------------------- the search over unordered chunks
//
// TE_NO_SORT=1: every pair of a chunk is examined in both passes.  The measure of what
// the ordered search (te_search.hip) prunes, and a check that does not depend on it.

template <int DY, int DX, int KP1, bool GENERIC>
__global__ void __launch_bounds__(kMaxWavesPerWG * 64) search_unordered_kernel(SearchArgs a)
{
    constexpr int D = 1 + DY + DX;
    constexpr int RW = (D + 1 + 3) & ~3;       // LDS row: D coordinates + radius, 16-byte aligned
    constexpr int SLOTS = 4;                   // candidates per lane in pass 2
    __shared__ __attribute__((aligned(16))) float rows[kMaxWavesPerWG * kWave * RW];
    const int lane = threadIdx.x & (kWave - 1);
    const int k = GENERIC ? a.k : KP1 - 1;

    const int nq = a.n_parts > 1 ? a.n_parts : 1;
    int qp = (int)(blockIdx.x % (unsigned)nq);   // this wave's queue
    int drained = 0;                              // queues found empty so far
    int last_ci = 0, last_lo = 0, last_hi = 0;    // the previous item's chunk and its item range
    unsigned long long work1 = 0, work2 = 0;      // pairs this wave evaluated in pass 1 / pass 2
    for (;;) {
        // ---- claim the next work item (wave-uniform)
        int q = 0;
        if (lane == 0)
            q = atomicAdd(a.counter + qp, 1);
        q = __builtin_amdgcn_readlane(q, 0);
        if (nq > 1) {
            q += uload_i(a.part_start + qp);
            if (q >= uload_i(a.part_start + qp + 1)) {
                if (++drained >= nq)
                    break;
                qp = qp + 1 == nq ? 0 : qp + 1;
                continue;
            }
        } else if (q >= a.n_items) {
            break;
        }
        // consecutive items of a queue are mostly blocks of one chunk
        if (q < last_lo || q >= last_hi) {
            last_ci = find_chunk(a.item_start, a.n_chunks, q);
            last_lo = uload_i(a.item_start + last_ci);
            last_hi = last_ci + 1 < a.n_chunks ? uload_i(a.item_start + last_ci + 1) : a.n_items;
        }
        const int ci = last_ci;
        ChunkDesc cd;
        {
            const char *w = reinterpret_cast<const char *>(a.chunks + ci);
            cd.tp = uload_l(reinterpret_cast<const int64_t *>(w + offsetof(ChunkDesc, tp)));
            cd.s = uload_l(reinterpret_cast<const int64_t *>(w + offsetof(ChunkDesc, s)));
            cd.geo = uload_l(reinterpret_cast<const int64_t *>(w + offsetof(ChunkDesc, geo)));
            cd.out = uload_l(reinterpret_cast<const int64_t *>(w + offsetof(ChunkDesc, out)));
            cd.pbase = uload_l(reinterpret_cast<const int64_t *>(w + offsetof(ChunkDesc, pbase)));
            cd.perm = uload_l(reinterpret_cast<const int64_t *>(w + offsetof(ChunkDesc, perm)));
            cd.n = uload_i(reinterpret_cast<const int32_t *>(w + offsetof(ChunkDesc, n)));
            cd.item0 = uload_i(reinterpret_cast<const int32_t *>(w + offsetof(ChunkDesc, item0)));
            cd.block0 = uload_i(reinterpret_cast<const int32_t *>(w + offsetof(ChunkDesc, block0)));
        }
        const int n = cd.n;
        const int blk = q - cd.item0 + cd.block0;
        const int r0 = blk * kWave;
        const Coords<DY, DX> cp(a.base, cd);

        // ---- pass 1: lane = reference i, candidates uniform
        const int i = r0 + lane;
        const bool valid = i < n;
        const int ii = valid ? i : n - 1;
        float ref[D];
#pragma unroll
        for (int m = 0; m < D; ++m)
            ref[m] = cp.p[m][ii];
        float best[KP1];
#pragma unroll
        for (int s = 0; s < KP1; ++s)
            best[s] = kInf;
        float thr = kInf;

        // current k+1-th distance of this lane: a candidate can only enter the
        // list if its joint distance is strictly below it
        auto cur = [&]() { return GENERIC ? thr : best[KP1 - 1]; };
        auto visit = [&](const float (&c)[D]) {
            const PairDist<DY, DX> d = pair_dist<DY, DX>(ref, c);
            const float dj = fmaxf(d.t, fmaxf(d.p, d.s));
            if (ballot(dj < cur())) {
                keep_branch();
                insert_sorted<KP1>(best, dj);
                if (GENERIC)
                    thr = kth<KP1, GENERIC>(best, k);
            }
        };
        // four consecutive candidates j..j+3 (scalar loads, one per coordinate)
        auto load4 = [&](int j, float (&c)[4][D]) {
            const uint32_t off = (uint32_t)j * 4u;
#pragma unroll
            for (int m = 0; m < D; ++m) {
                const f4v v = uload4_at(cp.p[m], off);
                c[0][m] = v.x;
                c[1][m] = v.y;
                c[2][m] = v.z;
                c[3][m] = v.w;
            }
        };
        // Four candidates at once: their distances are independent, and a
        // candidate that is not below the current k+1-th distance leaves the list
        // unchanged when inserted (med3 / min network), so one wave-wide test of
        // the group's smallest distance decides whether any insertion is needed,
        // and a test per candidate skips the insertions no lane needs.
        auto visit_group = [&](const float (&c)[4][D]) {
            float dj[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const PairDist<DY, DX> d = pair_dist<DY, DX>(ref, c[u]);
                dj[u] = fmaxf(d.t, fmaxf(d.p, d.s));
            }
            const float m = fminf(fminf(dj[0], dj[1]), fminf(dj[2], dj[3]));
            if (ballot(m < cur())) {
                keep_branch();
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (ballot(dj[u] < cur())) {
                        keep_branch();
                        insert_sorted<KP1>(best, dj[u]);
                        if (GENERIC)
                            thr = kth<KP1, GENERIC>(best, k);
                    }
            }
        };
        auto visit4 = [&](int j) {
            float c[4][D];
            load4(j, c);
            visit_group(c);
        };
        auto visit1 = [&](int j) {
            float c[D];
#pragma unroll
            for (int m = 0; m < D; ++m)
                c[m] = uload(cp.p[m] + j);
            visit(c);
        };
        const unsigned long long pass1_pairs = (unsigned long long)n * (unsigned long long)min(kWave, n - r0);
        int j = 0;
        for (; j + 4 <= n; j += 4)
            visit4(j);
        for (; j < n; ++j)
            visit1(j);
        // k+1-th smallest including self (distance 0) = k-th neighbour without self
        const float eps = cur();

        // ---- pass 2: lane = candidate, references uniform
        // Each lane parks its reference row (coordinates, then the radius) in
        // this wave's LDS rows; the counting loop reads them back as
        // wave-wide broadcasts, so a reference costs no SALU address work.
        float *myrows = rows + (threadIdx.x / kWave) * (kWave * RW);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int m = 0; m < D; ++m)
            myrows[lane * RW + m] = ref[m];
        myrows[lane * RW + D] = eps;
        __builtin_amdgcn_wave_barrier();

        const int nref = min(kWave, n - r0);
        uint32_t accP = 0, accTP = 0, accPS = 0;
        unsigned long long evaluated2 = 0;                // candidate-reference pairs examined in pass 2
        for (int t0 = 0; t0 < n; t0 += kWave * SLOTS) {
            float cand[SLOTS][D];
#pragma unroll
            for (int sl = 0; sl < SLOTS; ++sl) {
                const int idx = t0 + sl * kWave + lane;
                const bool ok = idx < n;
                // in-bounds load, lanes past the range masked below
                const uint32_t ic4 = (uint32_t)(ok ? idx : n - 1) * 4u;
#pragma unroll
                for (int m = 0; m < D; ++m) {
                    const float v = vload_at(cp.p[m], ic4);
                    cand[sl][m] = ok ? v : kInf;
                }
            }
            uint32_t tP = 0, tTP = 0, tPS = 0;
            evaluated2 += (unsigned long long)nref * (unsigned long long)min(kWave * SLOTS, n - t0);
            auto read_row = [&](int r, f4v (&row)[RW / 4]) {
                const f4v *rowv = reinterpret_cast<const f4v *>(myrows + r * RW);
#pragma unroll
                for (int v = 0; v < RW / 4; ++v)
                    row[v] = rowv[v];
            };
            auto count_ref = [&](const f4v (&row)[RW / 4], int r) {
                float rr[RW];
#pragma unroll
                for (int v = 0; v < RW / 4; ++v) {
                    rr[4 * v + 0] = row[v].x;
                    rr[4 * v + 1] = row[v].y;
                    rr[4 * v + 2] = row[v].z;
                    rr[4 * v + 3] = row[v].w;
                }
                const float er = rr[D];
                uint32_t sP = 0, sTP = 0, sPS = 0;
#pragma unroll
                for (int sl = 0; sl < SLOTS; ++sl) {
                    const PairDist<DY, DX> d = pair_dist_row<DY, DX, RW>(rr, cand[sl]);
                    const uint64_t mT = ballot(d.t < er);
                    const uint64_t mP = ballot(d.p < er);
                    const uint64_t mS = ballot(d.s < er);
                    sP += (uint32_t)__builtin_popcountll(mP);
                    sTP += (uint32_t)__builtin_popcountll(mP & mT);
                    sPS += (uint32_t)__builtin_popcountll(mP & mS);
                }
                tP = writelane(tP, sP, r);
                tTP = writelane(tTP, sTP, r);
                tPS = writelane(tPS, sPS, r);
            };
            for (int r = 0; r < nref; ++r) {
                f4v ra[RW / 4];
                read_row(r, ra);
                count_ref(ra, r);
            }
            accP += tP;
            accTP += tTP;
            accPS += tPS;
        }
        // self is at distance 0 in every space: counted iff eps > 0
        const uint32_t self = eps > 0.0f ? 1u : 0u;
        const int nP = (int)(accP - self), nTP = (int)(accTP - self), nPS = (int)(accPS - self);

        // ---- per-point digamma terms of eq. 9, summed over the item in fixed order
        double term = 0.0;
        if (valid)
            term = psi_of_count(nP) - psi_of_count(nTP) - psi_of_count(nPS);
        const double sum = wave_sum(term);
        if (lane == 0)
            a.partial[cd.pbase + blk] = sum;
        work1 += pass1_pairs;
        work2 += evaluated2;
        if (a.lte_out != nullptr && cd.out >= 0 && valid) {
            int o = (cd.perm >= 0) ? order_at(a.perm_base + cd.perm, n, i) : i;
            if (o < 0 || o >= n)
                o = i;
            a.lte_out[cd.out + o] = psi_of_count(k - 1) + term;
        }
        if (a.eps_out != nullptr && cd.out >= 0 && valid) {
            // per-point outputs go to the point's index before sorting
            int o = (cd.perm >= 0) ? order_at(a.perm_base + cd.perm, n, i) : i;
            if (o < 0 || o >= n)         // keep writes inside the chunk's output range regardless
                o = i;
            a.eps_out[cd.out + o] = eps;
            a.cnt_out[cd.out + o] = nP;
            a.cnt_out[a.cnt_stride + cd.out + o] = nTP;
            a.cnt_out[2 * a.cnt_stride + cd.out + o] = nPS;
        }
    }
    // measurement: one pair of counter updates per wave, after its last item
    if (a.work != nullptr && lane == 0) {
        atomicAdd(a.work, work1);
        atomicAdd(a.work + 1, work2);
        atomicAdd(a.work + 2, work1);
        atomicAdd(a.work + 3, work2);
    }
}

// ------------------------------------------------------------ small kernels

// Uniform [0, 1) floats from a counter hash (SplitMix64 finaliser); synthetic
// data for launch-shape tuning only.
__global__ void fill_uniform_kernel(float *p, int64_t n, uint64_t seed)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    uint64_t z = seed + (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    p[i] = (float)(z >> 40) * (1.0f / 16777216.0f);
}

__global__ void fill_i32_kernel(int32_t *p, int32_t v, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        p[i] = v;
}

// Bound by the gathers through the order map (100 windows of 5 000 points: 18.1 us with the boxes, 16.4 us
// without boxes and with a map of one sorted coordinate; 30 x 101 chunks, 1.0 GB written: 1.29 and 1.31 ms).
// One wave per block of 64 points at a time: the block's coordinates gathered through the order
// map, and with the window's first target block the block's box (target-past coordinates; the
// current source sample, which shuffles with the source, stays unbounded).
__global__ void embed_kernel(const float *__restrict__ x, const float *__restrict__ y,
                             const int32_t *__restrict__ perms, int32_t *sigma, uint64_t *scratch,
                             const int32_t *__restrict__ u_dev, const EmbedTask *__restrict__ tasks,
                             float *__restrict__ base, int R, int T, int d_y, int d_x, int tau, int u, int cond,
                             int32_t *err)
{
    const EmbedTask tk = tasks[blockIdx.x];
    const int n = tk.n;
    // source delay of this block: the launch's, the task's own, or one chosen on the device
    if (tk.u > 0)
        u = tk.u;
    if (tk.u_slot > 0 && u_dev != nullptr)
        u = u_dev[tk.u_slot - 1];
    // the host checks every delay against the window starts; keep reads in bounds regardless
    const bool u_ok = u >= 1 && tk.w - u - (d_x - 1) * tau >= 0 && tk.w + tk.W - u <= T;
    const int64_t pr = (int64_t)tk.pair * R;
    const int lane = threadIdx.x & (kWave - 1);
    const int nb = (n + kWave - 1) / kWave;
    float *box = nullptr;
    if (tk.box == 0)
        box = reinterpret_cast<float *>(sigma + tk.sig + box_words_behind_map(n));
    else if (tk.box > 0)
        box = reinterpret_cast<float *>(scratch + (int64_t)(tk.box - 1) * kBoxScratchUnit);
    bool bad = false;
    for (int qb = blockIdx.y * blockDim.x + (threadIdx.x - lane); qb < n; qb += blockDim.x * gridDim.y) {
        const bool ok = qb + lane < n;
        const int q = ok ? qb + lane : n - 1;
        // position q of the (ordered) chunk holds window point qo = r W + (t' - w)
        int qo = q;
        if (tk.sig >= 0) {
            qo = order_at(sigma + tk.sig, n, q);
            if (qo < 0 || qo >= n) {   // cannot happen for maps made by order_kernel; keep reads in bounds
                bad = true;
                qo = q;
            }
        }
        const int r = qo / tk.W;
        const int t = tk.w + (qo - r * tk.W);
        int rs = r;
        if (tk.perm >= 0) {
            rs = perms[tk.perm + r];
            if (rs < 0 || rs >= tk.Rc) {   // caller error; keep reads in bounds
                bad = true;
                rs = r;
            }
        }
        const float *yr = y + (pr + r) * T;
        const float *xr = x + (pr + rs) * T;
        if (tk.tp >= 0) {
            const float v0 = yr[t];
            bad |= !isfinite(v0);
            if (ok)
                base[tk.tp + q] = v0;
            for (int m = 0; m < d_y; ++m) {
                const float v = yr[t - 1 - m * tau];
                bad |= !isfinite(v);
                if (ok)
                    base[tk.tp + (int64_t)(1 + m) * n + q] = v;
                if (box != nullptr) {
                    float lo, hi;
                    wave_box(v, &lo, &hi);
                    if (lane == 0) {
                        box[(int64_t)(2 * m) * nb + qb / kWave] = lo;
                        box[(int64_t)(2 * m + 1) * nb + qb / kWave] = hi;
                    }
                }
            }
        }
        bad |= !u_ok;
        if (cond && tk.tp >= 0) {
            // the current source sample x_t joins the conditioning set: it is the last
            // target-past row of this chunk's own target block (it follows the shuffle)
            const float v = xr[t];
            bad |= !isfinite(v);
            if (ok)
                base[tk.tp + (int64_t)(1 + d_y) * n + q] = v;
            if (box != nullptr && lane == 0) {
                box[(int64_t)(2 * d_y) * nb + qb / kWave] = -kInf;
                box[(int64_t)(2 * d_y + 1) * nb + qb / kWave] = kInf;
            }
        }
        for (int m = 0; m < d_x; ++m) {
            const float v = u_ok ? xr[t - u - m * tau] : 0.0f;
            bad |= !isfinite(v);
            if (ok)
                base[tk.s + (int64_t)m * n + q] = v;
        }
    }
    if (bad)
        atomicOr(err, 1);
}

// One bitonic compare-exchange pass with stride jj inside stage kk over the
// len elements of A (LDS tile or global array).  offset: global index of A[0],
// so the sort direction is that of the full network.  Workgroup-wide: every
// thread takes pairs across the whole range.
__device__ __forceinline__ void bitonic_pass(uint64_t *A, int len, int kk, int jj, int offset)
{
    for (int t = threadIdx.x; t < len; t += blockDim.x) {
        const int i = t;
        const int l = i ^ jj;
        if (l > i) {
            const uint64_t u0 = A[i], u1 = A[l];
            const bool up = ((offset + i) & kk) == 0;
            if ((u0 > u1) == up) {
                A[i] = u1;
                A[l] = u0;
            }
        }
    }
}

// All passes of stage kk with stride jj < seg, for an LDS array split into
// seg-sized segments of which each wave owns one (or several): partners of
// strides below seg lie in the same segment, so a wave runs these passes back
// to back without workgroup barriers (LDS accesses of one wave complete in order).
__device__ __forceinline__ void bitonic_wave_passes(uint64_t *A, int len, int kk, int jstart, int seg, int offset)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int nwaves = blockDim.x / kWave;
    for (int s0 = wave * seg; s0 < len; s0 += nwaves * seg) {
        for (int jj = jstart; jj > 0; jj >>= 1) {
            for (int t = lane; t < seg; t += kWave) {
                const int i = s0 + t;
                const int l = i ^ jj;
                if (l > i) {
                    const uint64_t u0 = A[i], u1 = A[l];
                    const bool up = ((offset + i) & kk) == 0;
                    if ((u0 > u1) == up) {
                        A[i] = u1;
                        A[l] = u0;
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
}

// Full bitonic network over len (power of two) keys in LDS; offset as above.
// Strides of at least one wave segment run workgroup-wide with a barrier after
// each pass; the smaller strides of a stage run wave-locally.
__device__ void bitonic_lds(uint64_t *A, int len, int kk_first, int kk_last, int offset)
{
    const int nwaves = blockDim.x / kWave;
    const int seg = max(2, len / nwaves);        // keys per wave segment
    for (int kk = kk_first; kk <= kk_last; kk <<= 1) {
        int jj = kk >> 1;
        for (; jj >= seg; jj >>= 1) {
            bitonic_pass(A, len, kk, jj, offset);
            __syncthreads();
        }
        if (jj > 0) {
            bitonic_wave_passes(A, len, kk, jj, seg, offset);
            __syncthreads();
        }
    }
}

// First block of the slab that block `leaf` of nl lies in after `levels` cuts.
__device__ __forceinline__ int slab_start(int leaf, int nl, int nd, int levels)
{
    int first = 0, cnt = nl;
    for (int j = 0; j < levels; ++j) {
        const int s = slab_count(cnt, nd - j);
        // slab i of the run holds its blocks [cnt i / s, cnt (i + 1) / s)
        const int i = (int)(((int64_t)s * (leaf - first + 1) - 1) / cnt);
        const int a = (int)((int64_t)cnt * i / s), b = (int)((int64_t)cnt * (i + 1) / s);
        first += a;
        cnt = b - a;
    }
    return first;
}

// Whether cutting at level m leaves every slab of nl blocks whole: its sort would be for nothing.
__device__ __forceinline__ bool idle_level(int nl, int nd, int m)
{
    int cnt = nl;
    for (int j = 0; j < m; ++j) {
        const int s = slab_count(cnt, nd - j);
        cnt = (cnt + s - 1) / s;
    }
    return m + 1 < nd && slab_count(cnt, nd - m) == 1;
}

// Target-past coordinate m of point i of a task's search space.
struct CoordSource {
    const float *y, *pts;
    int64_t ld;
    int R, T, tau;
    __device__ __forceinline__ float at(const SortTask &tk, int i, int m) const
    {
        if (tk.mode != 0)
            return pts[tk.key_off + (int64_t)m * ld + i];
        const int r = i / tk.W;
        const int t = tk.w + (i - r * tk.W);
        return y[((int64_t)tk.pair * R + r) * T + t - 1 - m * tau];
    }
};

constexpr int kOrderThreads = 1024;
constexpr int kOrderWaves = kOrderThreads / kWave;
constexpr int kOrderEach = kSlabMax / kOrderThreads;   // points per thread at most

// Smallest and largest of the workgroup's values (red: 2 x kOrderWaves words of LDS).
__device__ __forceinline__ void block_range(uint32_t &lo, uint32_t &hi, uint32_t *red)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint32_t a = ~wave_max_u32(~lo), b = wave_max_u32(hi);
    if (lane == 0) {
        red[w] = a;
        red[kOrderWaves + w] = b;
    }
    __syncthreads();
    lo = ~wave_max_u32(~red[lane & (kOrderWaves - 1)]);
    hi = wave_max_u32(red[kOrderWaves + (lane & (kOrderWaves - 1))]);
    __syncthreads();
}

// Right shift that fits the range hi - lo into `bits` bits.
__device__ __forceinline__ int code_shift(uint32_t lo, uint32_t hi, int bits)
{
    return max(0, 32 - bits - (hi == lo ? 32 : __builtin_clz(hi - lo)));
}

// Lanes of the wave that hold the same BITS-bit digit as this one (inactive lanes hold none).
template <int BITS>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool active)
{
    const uint64_t act = ballot(active);
    uint32_t lo = (uint32_t)act, hi = (uint32_t)(act >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const uint32_t one = (uint32_t)((int32_t)(d << (31 - b)) >> 31);   // all ones where the bit is set
        const uint64_t mb = ballot(one != 0);
        lo &= ~((uint32_t)mb ^ one);
        hi &= ~((uint32_t)(mb >> 32) ^ one);
    }
    return (uint64_t)hi << 32 | lo;
}

__device__ __forceinline__ int rank_in(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Exclusive scan of cnt[w][d] over (d, w) in that order, in place, for DIGITS <= kOrderThreads
// digits and kOrderWaves waves: where each wave's elements of a digit go.  part: kOrderWaves words.
template <int DIGITS>
__device__ __forceinline__ void scan_digits(uint32_t *cnt, uint32_t *part)
{
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    uint32_t c[kOrderWaves], own = 0;
    if (t < DIGITS)
#pragma unroll
        for (int v = 0; v < kOrderWaves; ++v) {
            c[v] = cnt[v * DIGITS + t];
            own += c[v];
        }
    const uint32_t inc = wave_scan(own);                  // inclusive
    if (lane == kWave - 1)
        part[w] = inc;
    __syncthreads();
    if (t < DIGITS) {
        uint32_t base = inc - own;
        for (int v = 0; v < w; ++v)
            base += part[v];
#pragma unroll
        for (int v = 0; v < kOrderWaves; ++v) {
            cnt[v * DIGITS + t] = base;
            base += c[v];
        }
    }
    __syncthreads();
}

// Ordering, part 1 of 2, for spaces above kSlabMax points (and up to kMaxSlabs times as many): one
// workgroup cuts the space into
// order_slabs() slabs of whole blocks along the first target-past coordinate.  The coordinate
// is coded in 15 bits (its orderable image less the smallest, shifted to fit, so the code keeps
// at least the sign, the exponent and six bits of the mantissa, and everything where the values
// span little); the codes' histogram gives the code in which each cut falls.  A stable counting
// sort by the runs between those codes then puts every point on its side of every cut (points of
// a cut's own code by index), and leaves the point indices of each slab in index order in the map.
// The codes live behind the 16-bit map or in the key scratch, where the boxes will be written later.
// Bound by the latency of one workgroup's passes.  With order_kernel 113 us for one window of 48 000
// points and 53 us for five of 10 500; a bitonic sort by the first coordinate alone took 1 156 and 215 us.
constexpr int kCodeBits = 15;
constexpr int kClasses = 128;          // runs between cuts: 2 (kMaxSlabs - 1) + 1 at most

// Where a code's count is kept: rotated within its group of 32, so that threads which walk a group
// each read different banks (in code order a wave's reads all fall in one: 42 instead of 32 us for five
// windows of 10 500 points).
__device__ __forceinline__ uint32_t code_slot(uint32_t c) { return (c & ~31u) | ((c + (c >> 5)) & 31u); }

__global__ void __launch_bounds__(kOrderThreads) split_kernel(CoordSource src, const SortTask *__restrict__ tasks,
                                                              int32_t *sigma, uint64_t *scratch, int d_y)
{
    __shared__ uint32_t hist[1 << kCodeBits];             // code counts; then each code's class
    __shared__ uint32_t cnt[kOrderWaves * kClasses];
    __shared__ uint32_t part[2 * kOrderWaves];
    __shared__ int32_t cut_code[kMaxSlabs];
    const SortTask tk = tasks[blockIdx.x];
    const int n = tk.n, nd = tk.nd > 0 ? tk.nd : d_y;
    const int slabs = order_slabs(n, nd);                 // at least two: the launch has no other tasks
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const int nl = (n + kWave - 1) / kWave;
    int32_t *map = sigma + tk.sig;
    uint16_t *code = n <= kSortLds ? reinterpret_cast<uint16_t *>(map) + n
                                   : reinterpret_cast<uint16_t *>(scratch + tk.scratch);
    for (int i = t; i < (1 << kCodeBits); i += kOrderThreads)
        hist[i] = 0;
    for (int i = t; i < kOrderWaves * kClasses; i += kOrderThreads)
        cnt[i] = 0;
    // eight loads in flight per thread: a workgroup alone on its CU waits for each round of them
    constexpr int U = 8;
    uint32_t lo = ~0u, hi = 0;
    for (int i0 = t; i0 < n; i0 += U * kOrderThreads) {
        uint32_t o[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            o[u] = orderable(src.at(tk, min(i0 + u * kOrderThreads, n - 1), 0));
#pragma unroll
        for (int u = 0; u < U; ++u) {
            lo = min(lo, o[u]);
            hi = max(hi, o[u]);
        }
    }
    block_range(lo, hi, part);
    const int shift = code_shift(lo, hi, kCodeBits);
    for (int i0 = t; i0 < n; i0 += U * kOrderThreads) {
        uint32_t o[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            o[u] = orderable(src.at(tk, min(i0 + u * kOrderThreads, n - 1), 0));
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kOrderThreads;
            if (i < n) {
                const uint32_t c = code_slot((o[u] - lo) >> shift);
                code[i] = (uint16_t)c;
                atomicAdd(&hist[c], 1u);
            }
        }
    }
    __syncthreads();
    // thread t owns 32 consecutive codes: the code of each cut, then the class of every code
    constexpr int kOwn = (1 << kCodeBits) / kOrderThreads;
    uint32_t own = 0;
    for (int e = 0; e < kOwn; ++e)
        own += hist[code_slot(t * kOwn + e)];
    const uint32_t inc = wave_scan(own);                  // inclusive
    if (lane == kWave - 1)
        part[w] = inc;
    __syncthreads();
    uint32_t before = inc - own;
    for (int v = 0; v < w; ++v)
        before += part[v];
    if (own > 0) {
        // cuts whose rank lies in [before, before + own)
        uint32_t cum = before;
        int e = 0;
        for (int s = 1; s < slabs; ++s) {
            const uint32_t rank = (uint32_t)slab_first(nl, slabs, s) * kWave;
            if (rank < before || rank >= before + own)
                continue;
            while (cum + hist[code_slot(t * kOwn + e)] <= rank)
                cum += hist[code_slot(t * kOwn + e++)];
            cut_code[s] = t * kOwn + e;
        }
    }
    __syncthreads();
    {
        int s = 1, below = 0;                             // distinct cut codes below this thread's codes
        while (s < slabs && cut_code[s] < t * kOwn) {
            below += (s == 1 || cut_code[s] != cut_code[s - 1]);
            ++s;
        }
        for (int e = 0; e < kOwn; ++e) {
            const int c = t * kOwn + e;
            const bool cut = s < slabs && cut_code[s] == c;
            hist[code_slot(c)] = (uint32_t)(2 * below + (cut ? 1 : 0));
            if (cut) {
                ++below;
                while (s < slabs && cut_code[s] == c)
                    ++s;
            }
        }
    }
    __syncthreads();
    // stable counting sort by class: wave w takes a contiguous run of points
    const int run = ((n + kOrderThreads - 1) / kOrderThreads) * kWave;
    const int i1 = min(n, (w + 1) * run);
    for (int i0 = w * run + lane; i0 < i1; i0 += U * kWave) {
        uint32_t c[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            c[u] = code[min(i0 + u * kWave, n - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kWave < i1)
                atomicAdd(&cnt[w * kClasses + hist[c[u]]], 1u);
    }
    __syncthreads();
    scan_digits<kClasses>(cnt, part);
    for (int j0 = w * run; j0 < i1; j0 += U * kWave) {
        uint32_t cc[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            cc[u] = code[min(j0 + u * kWave + lane, n - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = j0 + u * kWave + lane;
            const bool ok = i < i1;
            const uint32_t c = ok ? hist[cc[u]] : 0u;
            const uint64_t m = match_digit<7>(c, ok);
            if (ok) {
                const int r = rank_in(m);
                const uint32_t at = cnt[w * kClasses + c] + (uint32_t)r;
                if (n <= kSortLds)
                    reinterpret_cast<uint16_t *>(map)[at] = (uint16_t)i;
                else
                    map[at] = i;
                __builtin_amdgcn_wave_barrier();
                if (r == 0)
                    cnt[w * kClasses + c] = at + (uint32_t)__builtin_popcountll(m);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// Ordering, part 2 of 2: workgroup (task, slab) orders one slab (a space of up to kSlabMax points
// whole) so that its blocks of 64 consecutive points are compact in the target past: sorted by a
// coordinate and cut into slabs of whole blocks, each slab sorted by the next coordinate and cut,
// and so on; the last coordinate orders the points of the last slabs.  Level m sorts by (slab,
// coordinate m) with stable radix passes of 8 bits in LDS: 16 bits of the coordinate, coded as in
// split_kernel, and the slab.  Points of equal keys keep the order of the level before, so the
// order is a function of the data alone.  A pass gives each wave a contiguous run of the points;
// lanes of equal digits find their ranks by ballots, the waves' digit counts are scanned once.
// Any order is correct (the boxes are taken from the points); this one is the same on every path.
// Bound by LDS latency: 18.8 us for one window of 2 000 points in two coordinates, 49 us for 100 windows
// of 5 000 in three; a radix sort by the first coordinate alone took 19.6 and 30.6 us, and the search
// behind it 128 and 1 238 us against 36 and 624 us.
template <bool LIST>                       // slabs of larger spaces among the tasks: their points listed in LDS
__global__ void __launch_bounds__(kOrderThreads) order_kernel(CoordSource src, const SortTask *__restrict__ tasks,
                                                              int32_t *sigma, int d_y, int n_cut, int per_cut,
                                                              int64_t first_wg)
{
    __shared__ struct {
        uint32_t key[kSlabMax];
        uint32_t cnt[kOrderWaves * 256];
        uint32_t part[2 * kOrderWaves];
        uint16_t loc[kSlabMax];
        uint8_t slab[kSlabMax / kWave];
    } sh;
    __shared__ uint32_t list[LIST ? kSlabMax : 1];
    // per_cut workgroups for each of the n_cut largest spaces, one for each of the others
    const int64_t wg = first_wg + blockIdx.x, cut_wgs = (int64_t)n_cut * per_cut;
    const SortTask tk = tasks[wg < cut_wgs ? wg / per_cut : n_cut + (wg - cut_wgs)];
    const int slab = wg < cut_wgs ? (int)(wg % per_cut) : 0;
    const int nd = tk.nd > 0 ? tk.nd : d_y;
    const int slabs = order_slabs(tk.n, nd);
    if (slab >= slabs)
        return;
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const int nl_all = (tk.n + kWave - 1) / kWave;
    const int first = slab_first(nl_all, slabs, slab);
    const int base = first * kWave;
    const int n = min(tk.n, slab_first(nl_all, slabs, slab + 1) * kWave) - base;
    const int nl = (n + kWave - 1) / kWave;
    int32_t *map = sigma + tk.sig;
    uint16_t *map16 = reinterpret_cast<uint16_t *>(map);
    const int level0 = slabs > 1 && nd > 1 ? 1 : 0;       // the slabs were cut along coordinate 0
    const int each = (n + kOrderThreads - 1) / kOrderThreads;
    if (nl_all == 1) {                                    // one block: any order will do
        if (t < n)
            map16[t] = (uint16_t)t;
        return;
    }
    const bool listed = LIST && slabs > 1;
    if (listed)
        for (int i = t; i < n; i += kOrderThreads)
            list[i] = tk.n <= kSortLds ? (uint32_t)map16[base + i] : (uint32_t)map[base + i];
    for (int i = t; i < n; i += kOrderThreads)
        sh.loc[i] = (uint16_t)i;
    __syncthreads();
    for (int m = level0; m < nd; ++m) {
        if (idle_level(nl, nd - level0, m - level0))
            continue;
        // keys of this level: wave w holds positions [w each 64, (w + 1) each 64)
        uint32_t key[kOrderEach];
        uint16_t loc[kOrderEach];
        uint32_t lo = ~0u, hi = 0;
#pragma unroll
        for (int e = 0; e < kOrderEach; ++e) {
            const int p = (w * each + e) * kWave + lane;
            if (e < each && p < n) {
                loc[e] = sh.loc[p];
                key[e] = orderable(src.at(tk, listed ? (int)list[loc[e]] : (int)loc[e], m));
                lo = min(lo, key[e]);
                hi = max(hi, key[e]);
            }
        }
        if (m > level0 && t < nl)
            sh.slab[t] = (uint8_t)slab_start(t, nl, nd - level0, m - level0);
        block_range(lo, hi, sh.part);
        if (lo == hi)                                     // nothing to sort by
            continue;
        const int shift = code_shift(lo, hi, 16);
#pragma unroll
        for (int e = 0; e < kOrderEach; ++e) {
            const int p = (w * each + e) * kWave + lane;
            if (e < each && p < n)
                key[e] = (key[e] - lo) >> shift | (m > level0 ? (uint32_t)sh.slab[p / kWave] << 16 : 0u);
        }
        const int bits = m > level0 ? 24 : 16;
        for (int bit = 0; bit < bits; bit += 8) {
            for (int i = t; i < kOrderWaves * 256; i += kOrderThreads)
                sh.cnt[i] = 0;
            __syncthreads();
            uint32_t at[kOrderEach];
#pragma unroll
            for (int e = 0; e < kOrderEach; ++e) {
                if (e >= each)
                    break;
                const bool ok = (w * each + e) * kWave + lane < n;
                const uint32_t d = (key[e] >> bit) & 255u;
                const uint64_t g = match_digit<8>(d, ok);
                if (ok) {
                    const int r = rank_in(g);
                    at[e] = sh.cnt[w * 256 + d] + (uint32_t)r;
                    __builtin_amdgcn_wave_barrier();
                    if (r == 0)
                        sh.cnt[w * 256 + d] = at[e] + (uint32_t)__builtin_popcountll(g);
                }
                __builtin_amdgcn_wave_barrier();
            }
            __syncthreads();
            scan_digits<256>(sh.cnt, sh.part);
#pragma unroll
            for (int e = 0; e < kOrderEach; ++e)
                if (e < each && (w * each + e) * kWave + lane < n) {
                    const uint32_t p = at[e] + sh.cnt[w * 256 + ((key[e] >> bit) & 255u)];
                    sh.key[p] = key[e];
                    sh.loc[p] = loc[e];
                }
            __syncthreads();
            if (bit + 8 < bits)
#pragma unroll
                for (int e = 0; e < kOrderEach; ++e) {
                    const int p = (w * each + e) * kWave + lane;
                    if (e < each && p < n) {
                        key[e] = sh.key[p];
                        loc[e] = sh.loc[p];
                    }
                }
        }
        __syncthreads();
    }
    for (int i = t; i < n; i += kOrderThreads) {
        const uint32_t o = listed ? list[sh.loc[i]] : (uint32_t)sh.loc[i];
        if (tk.n <= kSortLds)
            map16[base + i] = (uint16_t)o;
        else
            map[base + i] = (int32_t)o;
    }
}

// Ordering, part 1 of 2, for spaces above kMaxSlabs x kSlabMax points: the map sorted by the first
// target-past coordinate, which cuts it into slabs for order_kernel.  A bitonic network over npad = 2^k
// keys (coordinate, index; padding keys sort last) in global scratch: the stages up to kSortLds keys in
// the LDS of a workgroup per tile of that many, then per stage a launch for each wider stride and one for
// the strides inside the tiles.  Bound by the passes over global memory: all of it in one workgroup took
// 30.6 ms for 600 000 points (a call with d_y = 2 36.2 ms, now 5.7).
__global__ void __launch_bounds__(kOrderThreads) whole_tiles_kernel(CoordSource src, const SortTask *__restrict__ tasks,
                                                                    uint64_t *scratch)
{
    __shared__ uint64_t lds[kSortLds];
    const SortTask tk = tasks[blockIdx.y];
    const int64_t t0 = (int64_t)blockIdx.x * kSortLds;
    if (t0 >= tk.npad)
        return;
    uint64_t *A = scratch + tk.scratch + t0;
    for (int x = threadIdx.x; x < kSortLds; x += kOrderThreads) {
        const int i = (int)t0 + x;
        lds[x] = i < tk.n ? (uint64_t)orderable(src.at(tk, i, 0)) << 32 | (uint32_t)i : ~0ull;
    }
    __syncthreads();
    bitonic_lds(lds, kSortLds, 2, kSortLds, (int)t0);
    for (int x = threadIdx.x; x < kSortLds; x += kOrderThreads)
        A[x] = lds[x];
}

// Stride jj >= kSortLds of stage kk.
__global__ void __launch_bounds__(256) whole_stride_kernel(const SortTask *__restrict__ tasks, uint64_t *scratch, int kk,
                                                           int jj)
{
    const SortTask tk = tasks[blockIdx.y];
    if (kk > tk.npad)
        return;
    uint64_t *A = scratch + tk.scratch;
    for (int p = blockIdx.x * 256 + threadIdx.x; p < tk.npad / 2; p += gridDim.x * 256) {
        const int i = (p & ~(jj - 1)) * 2 + (p & (jj - 1)), l = i + jj;
        const uint64_t u0 = A[i], u1 = A[l];
        if ((u0 > u1) == ((i & kk) == 0)) {
            A[i] = u1;
            A[l] = u0;
        }
    }
}

// The strides of stage kk inside the tiles; after a space's last stage the map.
__global__ void __launch_bounds__(kOrderThreads) whole_merge_kernel(const SortTask *__restrict__ tasks, int32_t *sigma,
                                                                    uint64_t *scratch, int kk)
{
    __shared__ uint64_t lds[kSortLds];
    const SortTask tk = tasks[blockIdx.y];
    const int64_t t0 = (int64_t)blockIdx.x * kSortLds;
    if (kk > tk.npad || t0 >= tk.npad)
        return;
    uint64_t *A = scratch + tk.scratch + t0;
    for (int x = threadIdx.x; x < kSortLds; x += kOrderThreads)
        lds[x] = A[x];
    __syncthreads();
    constexpr int seg = kSortLds / kOrderWaves;
    for (int jj = kSortLds >> 1; jj >= seg; jj >>= 1) {
        bitonic_pass(lds, kSortLds, kk, jj, (int)t0);
        __syncthreads();
    }
    bitonic_wave_passes(lds, kSortLds, kk, seg >> 1, seg, (int)t0);
    __syncthreads();
    for (int x = threadIdx.x; x < kSortLds; x += kOrderThreads) {
        if (kk < tk.npad)
            A[x] = lds[x];
        else if (t0 + x < tk.n)
            sigma[tk.sig + t0 + x] = (int32_t)(uint32_t)lds[x];
    }
}

__global__ void gather_kernel(const float *__restrict__ src, const GatherTask *__restrict__ tasks,
                              int32_t *sigma, uint64_t *scratch, float *__restrict__ dst, int D, int d_y)
{
    const GatherTask tk = tasks[blockIdx.x];
    const int n = tk.n;
    const int lane = threadIdx.x & (kWave - 1);
    const int nb = (n + kWave - 1) / kWave;
    float *box = nullptr;
    if (nb > 1)
        box = n <= kSortLds ? reinterpret_cast<float *>(sigma + tk.sig + box_words_behind_map(n))
                            : reinterpret_cast<float *>(scratch + (int64_t)tk.box * kBoxScratchUnit);
    for (int qb = blockIdx.y * blockDim.x + (threadIdx.x - lane); qb < n; qb += blockDim.x * gridDim.y) {
        const bool ok = qb + lane < n;
        const int q = ok ? qb + lane : n - 1;
        int o = order_at(sigma + tk.sig, n, q);
        if (o < 0 || o >= n)          // maps from order_kernel are permutations; keep reads in bounds regardless
            o = q;
        for (int m = 0; m < D; ++m) {
            const float v = src[tk.src + (int64_t)m * tk.ld + o];
            if (ok)
                dst[tk.dst + (int64_t)m * n + q] = v;
            if (box != nullptr && m >= 1 && m <= d_y) {
                float lo, hi;
                wave_box(v, &lo, &hi);
                if (lane == 0) {
                    box[(int64_t)(2 * (m - 1)) * nb + qb / kWave] = lo;
                    box[(int64_t)(2 * (m - 1) + 1) * nb + qb / kWave] = hi;
                }
            }
        }
    }
}

// ------------------------------------------------------ surrogate permutations

constexpr int kMaxPermTrials = 1 << 16;

// Copy mode: row i of the caller's permutations into the batch's permutation
// area.  Entries < rc must be a permutation of 0..rc-1 (one workgroup per row,
// an LDS bitmap records the values seen); entries rc..len-1 are the identity.
__global__ void take_perms_kernel(const int32_t *__restrict__ src, const PermTask *__restrict__ tasks,
                                  int32_t *__restrict__ dst, int32_t *err)
{
    __shared__ uint32_t seen[kMaxPermTrials / 32];
    const PermTask tk = tasks[blockIdx.x];
    const int rc = tk.rc;
    const bool too_big = rc > kMaxPermTrials || rc < 1;
    const int words = too_big ? 0 : (rc + 31) / 32;
    for (int w = threadIdx.x; w < words; w += blockDim.x)
        seen[w] = 0;
    __syncthreads();
    bool bad = too_big;
    if (!bad) {
        for (int r = threadIdx.x; r < rc; r += blockDim.x) {
            const int v = src[tk.src + r];
            if (v < 0 || v >= rc) {
                bad = true;
                dst[tk.dst + r] = r;          // keep later reads in bounds; the call reports the error
            } else {
                const uint32_t bit = 1u << (v & 31);
                if (atomicOr(&seen[v >> 5], bit) & bit)
                    bad = true;
                dst[tk.dst + r] = v;
            }
        }
    }
    for (int r = max(rc, 0) + threadIdx.x; r < tk.len; r += blockDim.x)
        dst[tk.dst + r] = r;
    if (bad)
        atomicOr(err, 2);
}

// Seeded mode.  The permutation of (pair p, point c, surrogate s) is drawn from
// the counter-based SplitMix64 generator (Steele, Lea and Flood 2014): output q
// of the stream with key K is mix(K + (q + 1) G), and K folds the identifiers
// into the seed, K = f(f(f(f(f(0x5EED5EED5EED5EED, seed), 77), p), c), s) with
// f(k, v) = mix(k + G v + 1).  Fisher-Yates from the top: for i = rc-1 down to 1,
// swap positions i and j_i, j_i uniform on 0..i.  Draw number t = rc-1-i takes its
// bound i + 1 and Lemire's multiply-and-reject rule on the high 32 bits w of an
// output: m = w (i + 1), j_i = m >> 32, rejected when (m mod 2^32) < 2^32 mod (i+1).
// Draws are made in rounds: in round one draw t takes output t; each later round
// gives the draws rejected so far, in draw order, the next unused outputs.
// The rejected draws (in one of 4 400 rows of 2 000 trials, one of 700 of 5 000) take their later
// rounds on one wave (redraw); the swaps are resolved in parallel (draw_perms_kernel), in rows of more
// than kDrawShared trials made in order by one lane (draw_long_perms_kernel).
constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;
constexpr int kDrawShared = 8192;         // 10 bytes of LDS per trial: 80 KB, one row per CU at most
constexpr int kDrawThreads = 256;
constexpr int kMaxRejects = 256;

__device__ __forceinline__ uint64_t mix64(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t fold_key(uint64_t k, uint64_t v) { return mix64(k + kGolden * v + 1ull); }

// Lemire's rule for bound s on output q of stream key: the draw, or -1 if rejected.
__device__ __forceinline__ int lemire_draw(uint64_t key, uint64_t q, uint32_t s)
{
    const uint32_t w = (uint32_t)(mix64(key + (q + 1ull) * kGolden) >> 32);
    const uint64_t m = (uint64_t)w * s;
    const uint32_t lo = (uint32_t)m;
    if (lo < s && lo < (0u - s) % s)
        return -1;
    return (int)(m >> 32);
}

__device__ __forceinline__ uint64_t row_key(uint64_t seed, const PermTask &tk)
{
    uint64_t key = 0x5EED5EED5EED5EEDull;
    key = fold_key(key, seed);
    key = fold_key(key, 77ull);
    key = fold_key(key, (uint64_t)(int64_t)tk.pair);
    key = fold_key(key, (uint64_t)(int64_t)tk.point);
    return fold_key(key, (uint64_t)(int64_t)tk.surr);
}

// The rejected draws of a row and what they draw in the end: draw t[f] gives j[f] for f < n.
struct Redrawn {
    int32_t n;                            // below 0: more rejected draws than the lists hold
    int32_t t[kMaxRejects], j[kMaxRejects];
};

// One wave: the later rounds of the npend draws listed, in any order, in pend[1].
__device__ void redraw(uint64_t key, int n, int npend, int32_t (&pend)[2][kMaxRejects], Redrawn &out)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t lanes_below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    if (npend > kMaxRejects) {
        if (lane == 0)
            out.n = -1;
        return;
    }
    // in draw order
    for (int l = lane; l < npend; l += kWave) {
        int rank = 0;
        for (int m = 0; m < npend; ++m)
            rank += pend[1][m] < pend[1][l];
        pend[0][rank] = pend[1][l];
    }
    // pending draws take the next unused outputs, in draw order
    uint64_t pos = (uint64_t)max(n - 1, 0);
    int nfix = 0, cur = 0;
    while (npend > 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int nnext = 0;
        for (int b0 = 0; b0 < npend; b0 += kWave) {
            const int l = b0 + lane;
            int t = 0, j = -1;
            if (l < npend) {
                t = pend[cur][l];
                j = lemire_draw(key, pos + (uint64_t)l, (uint32_t)(n - t));
            }
            const bool acc = l < npend && j >= 0;
            const bool rej = l < npend && j < 0;
            const uint64_t ma = ballot(acc), mr = ballot(rej);
            if (acc) {
                const int idx = nfix + __builtin_popcountll(ma & lanes_below);
                out.t[idx] = t;
                out.j[idx] = j;
            }
            if (rej)
                pend[cur ^ 1][nnext + __builtin_popcountll(mr & lanes_below)] = t;
            nfix += __builtin_popcountll(ma);
            nnext += __builtin_popcountll(mr);
        }
        pos += (uint64_t)npend;
        npend = nnext;
        cur ^= 1;
    }
    if (lane == 0)
        out.n = nfix;
}

// The swaps of a row of n trials, in order, by one wave's first lane.
__device__ void swap_row(int32_t *row, uint64_t key, int n, const Redrawn &fix)
{
    const int lane = threadIdx.x & (kWave - 1);
    for (int r = lane; r < n; r += kWave)
        row[r] = r;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane == 0) {
        for (int t = 0; t < n - 1; ++t) {
            const int i = n - 1 - t;
            int j = lemire_draw(key, (uint64_t)t, (uint32_t)(i + 1));
            if (j < 0)
                for (int f = 0; f < fix.n; ++f)
                    if (fix.t[f] == t)
                        j = fix.j[f];
            if (j < 0 || j > i)              // cannot happen: every rejected draw has a fix
                j = i;
            const int32_t vi = row[i], vj = row[j];
            row[i] = vj;
            row[j] = vi;
        }
    }
}

// Rows of more than kDrawShared trials, a wave each: the swaps in order, in the row itself (9 000 trials: 2 ms).
__global__ void __launch_bounds__(kWave) draw_long_perms_kernel(const PermTask *__restrict__ tasks,
                                                                int32_t *__restrict__ dst, uint64_t seed, int32_t *err)
{
    __shared__ int32_t rejected, pend[2][kMaxRejects];
    __shared__ Redrawn fix;
    const PermTask tk = tasks[blockIdx.x];
    const int n = tk.rc, lane = threadIdx.x;
    if (n <= kDrawShared)
        return;
    int32_t *row = dst + tk.dst;
    const bool too_big = n > kMaxPermTrials;
    for (int r = too_big ? lane : n + lane; r < tk.len; r += kWave)
        row[r] = r;
    if (too_big) {
        if (lane == 0)
            atomicOr(err, 2);
        return;
    }
    const uint64_t key = row_key(seed, tk);
    if (lane == 0)
        rejected = 0;
    __syncthreads();
    for (int t = lane; t < n - 1; t += kWave)
        if (lemire_draw(key, (uint64_t)t, (uint32_t)(n - t)) < 0) {
            const int l = atomicAdd(&rejected, 1);
            if (l < kMaxRejects)
                pend[1][l] = t;
        }
    __syncthreads();
    redraw(key, n, rejected, pend, fix);
    __syncthreads();
    if (fix.n < 0) {
        for (int r = lane; r < n; r += kWave)
            row[r] = r;
        if (lane == 0)
            atomicOr(err, 2);
        return;
    }
    swap_row(row, key, n, fix);
}

// One workgroup per row.  What position i holds in the end is what position j_i held when step i
// swapped them (steps run from i = n-1 down): the entry that the last earlier step i' > i with
// j_i' = j_i had put there, or j_i itself; step i' had put there what position i' held then, and so
// on.  With next(p) = the smallest step i > p with j_i = p, that is
//   a[i] = end(s) for s = the smallest step above i with j_s = j_i, or j_i if there is none,
// end(p) following next() to its end; a[0] = end(0).  The steps of equal j are chained by exchanges in
// LDS (in any order: only minima are taken from a chain), chains and paths being a few steps long.
// Bound by LDS latency: 500 rows of 5 000 / 8 192 trials 70 / 130 us a call, rejected draws among them (a
// row with one costs a microsecond more); one lane making a row's swaps in order 890 / 1 440 us.
__global__ void __launch_bounds__(kDrawThreads) draw_perms_kernel(const PermTask *__restrict__ tasks,
                                                                  int32_t *__restrict__ dst, uint64_t seed, int32_t *err)
{
    extern __shared__ __attribute__((aligned(16))) char draw_lds[];
    __shared__ int32_t rejected, pend[2][kMaxRejects];
    __shared__ Redrawn fix;
    constexpr uint16_t kEnd = 0xffff;
    const PermTask tk = tasks[blockIdx.x];
    const int n = tk.rc, tid = threadIdx.x;
    if (n > kDrawShared)                  // draw_long_perms_kernel
        return;
    int32_t *row = dst + tk.dst;
    for (int r = max(n, 0) + tid; r < tk.len; r += kDrawThreads)
        row[r] = r;
    if (n < 1) {
        if (tid == 0)
            atomicOr(err, 2);
        return;
    }
    const uint64_t key = row_key(seed, tk);
    int32_t *head = reinterpret_cast<int32_t *>(draw_lds);
    uint16_t *j = reinterpret_cast<uint16_t *>(head + n), *chain = j + n, *next = chain + n;
    if (tid == 0)
        rejected = 0;
    __syncthreads();
    for (int i = tid; i < n; i += kDrawThreads) {
        head[i] = kEnd;
        const int d = i > 0 ? lemire_draw(key, (uint64_t)(n - 1 - i), (uint32_t)(i + 1)) : 0;
        if (d < 0) {
            const int l = atomicAdd(&rejected, 1);
            if (l < kMaxRejects)
                pend[1][l] = n - 1 - i;
        }
        j[i] = (uint16_t)max(d, 0);
    }
    __syncthreads();
    if (rejected > 0) {
        if (tid < kWave)
            redraw(key, n, rejected, pend, fix);
        __syncthreads();
        if (fix.n < 0) {
            for (int r = tid; r < n; r += kDrawThreads)
                row[r] = r;
            if (tid == 0)
                atomicOr(err, 2);
            return;
        }
        for (int f = tid; f < fix.n; f += kDrawThreads)
            j[n - 1 - fix.t[f]] = (uint16_t)fix.j[f];
        __syncthreads();
    }
    for (int i = tid; i < n; i += kDrawThreads)
        if (i > 0)
            chain[i] = (uint16_t)atomicExch(&head[j[i]], i);
    __syncthreads();
    // the smallest step above i in the chain of position p
    auto above = [&](int p, int i) {
        int best = kEnd;
        for (int s = head[p]; s != kEnd; s = chain[s])
            best = s > i ? min(best, s) : best;
        return best;
    };
    for (int p = tid; p < n; p += kDrawThreads)
        next[p] = (uint16_t)above(p, p);
    __syncthreads();
    for (int i = tid; i < n; i += kDrawThreads) {
        const int p = i > 0 ? (int)j[i] : 0;
        int s = above(p, i), v = p;
        while (s != kEnd) {
            v = s;
            s = next[s];
        }
        row[i] = v;
    }
}

// p-value of window group g (eq. 10 test): the fraction of its n_surr surrogate
// estimates at or above the original (results [g][0] original, [g][1..] surrogates)
__device__ __forceinline__ double group_pvalue(const double *results, int g, int n_surr)
{
    const double *r = results + (int64_t)g * (n_surr + 1);
    int c = 0;
    for (int s = 1; s <= n_surr; ++s)
        c += r[s] >= r[0];
    return n_surr > 0 ? (double)c / (double)n_surr : __builtin_nan("");
}

__global__ void reduce_kernel(const ChunkDesc *__restrict__ chunks, int n_chunks,
                              const double *__restrict__ partial, int k, const int32_t *err,
                              double *results, int n_groups, int n_surr, double *__restrict__ pv,
                              int32_t *done, int32_t *err_out)
{
    // one wave per chunk: lane l sums items l, l + 64, ... in order, then a fixed
    // butterfly across the wave (the same order on every run and batch split)
    const int c = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    if (c < n_chunks) {
        const ChunkDesc cd = chunks[c];
        const int nb = (cd.n + kWave - 1) / kWave;
        double s = 0.0;
        for (int b = lane; b < nb; b += kWave)
            s += partial[cd.pbase + b];
        s = wave_sum(s);
        if (lane == 0) {
            double te = psi_of_count(k - 1) + s / (double)cd.n;
            if (*err != 0)
                te = __builtin_nan("");
            results[cd.result] = te;
        }
    }
    if (pv == nullptr)
        return;
    // the workgroup that finishes last (done counts finished workgroups, zero at
    // launch) computes every group's p-value and copies the error word behind them
    __shared__ int last;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0)
        last = atomicAdd(done, 1) == (int)gridDim.x - 1;
    __syncthreads();
    if (!last)
        return;
    __threadfence();
    const bool bad = *err != 0;
    for (int g = threadIdx.x; g < n_groups; g += blockDim.x)
        pv[g] = bad ? __builtin_nan("") : group_pvalue(results, g, n_surr);
    if (threadIdx.x == 0 && err_out != nullptr)
        *err_out = *err;
}

__global__ void pvalue_kernel(const double *__restrict__ results, int n_groups, int n_surr,
                              double *__restrict__ pv, const int32_t *err, int32_t *err_out)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g == 0 && err_out != nullptr)
        *err_out = *err;
    if (g >= n_groups)
        return;
    pv[g] = (err != nullptr && *err != 0) ? __builtin_nan("") : group_pvalue(results, g, n_surr);
}

// Delay reconstruction (eq. 5): per window group, the delay whose original
// estimate is largest (the first one in table order among equal maxima).
__global__ void argmax_u_kernel(const double *__restrict__ results, int n_groups, int n_u,
                                const int32_t *__restrict__ u_values, int32_t *__restrict__ u_sel)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n_groups)
        return;
    const double *r = results + (int64_t)g * n_u;
    int best = 0;
    for (int j = 1; j < n_u; ++j)
        if (r[j] > r[best])
            best = j;
    u_sel[g] = u_values[best];
}

// ------------------------------------------------------------- dispatch

typedef void (*search_fn)(SearchArgs);

search_fn pick_unordered(int d_y, int d_x, int k)
{
#define TE_CASE(A, B)             \
    if (d_y == A && d_x == B)     \
        return k != 4 ? search_unordered_kernel<A, B, kMaxK + 1, true> : search_unordered_kernel<A, B, 5, false>;
    TE_CASE(1, 1) TE_CASE(1, 2) TE_CASE(1, 3) TE_CASE(1, 4)
    TE_CASE(2, 1) TE_CASE(2, 2) TE_CASE(2, 3) TE_CASE(2, 4)
    TE_CASE(3, 1) TE_CASE(3, 2) TE_CASE(3, 3) TE_CASE(3, 4)
    TE_CASE(4, 1) TE_CASE(4, 2) TE_CASE(4, 3) TE_CASE(4, 4)
#undef TE_CASE
    return nullptr;
}

int occupancy(search_fn f, int waves_per_wg, size_t lds)
{
    int blocks = 0;
    if (!f || hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, f, kWave * waves_per_wg, lds) != hipSuccess)
        return 0;
    return blocks;
}

}  // namespace

// Device counters of evaluated pairs for the measurement hook (one copy per device):
// [0] pass-1 and [1] pass-2 (reference, candidate, chunk) triples, [2] and [3] the
// (reference, candidate) pairs whose shared coordinates were evaluated once for them.
__device__ unsigned long long g_work_counters[4];

unsigned long long *work_counters()
{
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_work_counters)) != hipSuccess)
        return nullptr;
    return static_cast<unsigned long long *>(p);
}

bool search_supported(int d_y, int d_x, int k, int slots)
{
    return pick_ordered(d_y, d_x, k, slots, false, 1).fn != nullptr;
}

// Resident workgroups per compute unit for the chosen search variant (0 if unknown).
int search_occupancy(int d_y, int d_x, int k, int slots, int waves_per_wg)
{
    const ordered_search s = pick_ordered(d_y, d_x, k, slots, false, waves_per_wg);
    return occupancy(s.fn, waves_per_wg, s.lds);
}

bool search_sets_supported(int d_y, int d_x, int k) { return pick_ordered(d_y, d_x, k, 4, true, 1).fn != nullptr; }

int search_sets_occupancy(int d_y, int d_x, int slots, int waves_per_wg)
{
    const ordered_search s = pick_ordered(d_y, d_x, 4, slots, true, waves_per_wg);
    return occupancy(s.fn, waves_per_wg, s.lds);
}

hipError_t launch_search(const SearchArgs &a, int d_y, int d_x, const SearchConfig &cfg, int grid_waves,
                         hipStream_t st)
{
    const int wpg = cfg.waves_per_wg;
    const int blocks = (grid_waves + wpg - 1) / wpg;
    ordered_search s{nullptr, 0};
    const int set_coords = a.set_first != nullptr ? 1 + d_y + set_variants(d_y, d_x) * d_x : 0;
    const int w = a.sorted && !cfg.timed ? waves_to_a_block(a.n_items, set_coords, a.k, a.n_parts > 1) : 0;
    if (w > 0) {
        s = pick_shared(d_y, d_x, a.k, a.set_first != nullptr, w);
        if (!s.fn)
            return hipErrorInvalidValue;
        hipLaunchKernelGGL(s.fn, dim3(a.n_items), dim3(kWave * w), s.lds, st, a);
        return hipGetLastError();
    }
    if (a.sorted)
        s = pick_ordered(d_y, d_x, a.k, cfg.slots, a.set_first != nullptr, wpg);
    else if (a.set_first == nullptr && a.k >= 1 && a.k <= kMaxK)
        s.fn = pick_unordered(d_y, d_x, a.k);
    if (!s.fn)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(s.fn, dim3(blocks), dim3(kWave * wpg), s.lds, st, a);
    return hipGetLastError();
}

hipError_t launch_fill_uniform(float *p, int64_t n, uint64_t seed, hipStream_t st)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(fill_uniform_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, seed);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t st)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

// Workgroups per task of the kernels that take a task's points 256 at a time: one round each while that
// leaves the launch small (its time is then one round's latency), else four or more.
static int point_parts(int n_tasks, int max_n)
{
    const int rounds = (max_n + 255) / 256;
    return std::max(1, std::min(1024, (int64_t)n_tasks * rounds <= 4096 ? rounds : (rounds + 3) / 4));
}

hipError_t launch_embed(const float *x, const float *y, const int32_t *perms, int32_t *sigma, uint64_t *scratch,
                        const int32_t *u_dev, const EmbedTask *tasks, int n_tasks, int max_n, float *base, int R,
                        int T, int d_y, int d_x, int tau, int u, int cond, int32_t *err, hipStream_t st)
{
    if (n_tasks <= 0)
        return hipSuccess;
    const int parts = point_parts(n_tasks, max_n);
    hipLaunchKernelGGL(embed_kernel, dim3(n_tasks, parts), dim3(256), 0, st, x, y, perms, sigma, scratch, u_dev, tasks, base,
                       R, T, d_y, d_x, tau, u, cond, err);
    return hipGetLastError();
}

hipError_t launch_argmax_u(const double *results, int n_groups, int n_u, const int32_t *u_values, int32_t *u_sel,
                           hipStream_t st)
{
    if (n_groups <= 0 || n_u <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(argmax_u_kernel, dim3((n_groups + 127) / 128), dim3(128), 0, st, results, n_groups, n_u,
                       u_values, u_sel);
    return hipGetLastError();
}

hipError_t launch_sort(const float *y, const float *pts, int64_t ld, const SortTask *tasks, const SortSizes &sizes,
                       int32_t *sigma, uint64_t *scratch, int R, int T, int d_y, int tau, hipStream_t st)
{
    const CoordSource src{y, pts, ld, R, T, tau};
    const dim3 block(kOrderThreads);
    if (sizes.n_cut == 0) {
        if (sizes.n_tasks > 0)
            hipLaunchKernelGGL(order_kernel<false>, dim3(sizes.n_tasks), block, 0, st, src, tasks, sigma, d_y, 0, 1,
                               (int64_t)0);
        return hipGetLastError();
    }
    if (sizes.n_cut > sizes.n_whole)
        hipLaunchKernelGGL(split_kernel, dim3(sizes.n_cut - sizes.n_whole), block, 0, st, src, tasks + sizes.n_whole,
                           sigma, scratch, d_y);
    if (sizes.n_whole > 0) {
        int64_t np = kSortLds;
        while (np < sizes.max_n)
            np *= 2;
        const dim3 tiles((unsigned)(np / kSortLds), sizes.n_whole);
        const dim3 strides((unsigned)std::min<int64_t>(8192, np / 2048), sizes.n_whole);
        hipLaunchKernelGGL(whole_tiles_kernel, tiles, block, 0, st, src, tasks, scratch);
        for (int64_t kk = 2 * kSortLds; kk <= np; kk *= 2) {
            for (int64_t jj = kk / 2; jj >= kSortLds; jj /= 2)
                hipLaunchKernelGGL(whole_stride_kernel, strides, dim3(256), 0, st, tasks, scratch, (int)kk, (int)jj);
            hipLaunchKernelGGL(whole_merge_kernel, tiles, block, 0, st, tasks, sigma, scratch, (int)kk);
        }
    }
    // the most slabs of any task: order_slabs grows with n
    int slabs = order_slabs(sizes.max_n, d_y > 0 ? d_y : 1);
    for (int nd = 2; d_y == 0 && nd <= 4; ++nd)
        slabs = std::max(slabs, order_slabs(sizes.max_n, nd));
    const int64_t wgs = (int64_t)sizes.n_cut * slabs + (sizes.n_tasks - sizes.n_cut);
    constexpr int64_t kGrid = 1 << 21;                    // a grid holds fewer than 2^32 threads
    for (int64_t w0 = 0; w0 < wgs; w0 += kGrid)
        hipLaunchKernelGGL(order_kernel<true>, dim3((unsigned)std::min(kGrid, wgs - w0)), block, 0, st, src, tasks, sigma,
                           d_y, sizes.n_cut, slabs, w0);
    return hipGetLastError();
}

hipError_t launch_gather(const float *src, const GatherTask *tasks, int n_tasks, int max_n, int32_t *sigma,
                         uint64_t *scratch, float *dst, int D, int d_y, hipStream_t st)
{
    if (n_tasks <= 0)
        return hipSuccess;
    const int parts = point_parts(n_tasks, max_n);
    hipLaunchKernelGGL(gather_kernel, dim3(n_tasks, parts), dim3(256), 0, st, src, tasks, sigma, scratch, dst, D, d_y);
    return hipGetLastError();
}

hipError_t launch_perms(const int32_t *src, const PermTask *tasks, int n_tasks, int max_rc, int32_t *dst,
                        uint64_t seed, int32_t *err, hipStream_t st)
{
    if (n_tasks <= 0)
        return hipSuccess;
    if (src != nullptr)
        hipLaunchKernelGGL(take_perms_kernel, dim3(n_tasks), dim3(256), 0, st, src, tasks, dst, err);
    else {
        hipLaunchKernelGGL(draw_perms_kernel, dim3(n_tasks), dim3(kDrawThreads),
                           (size_t)10 * std::max(0, std::min(max_rc, kDrawShared)) + 16, st, tasks, dst, seed, err);
        // apart, so that the rows that need no LDS do not wait for a CU's LDS each
        if (max_rc > kDrawShared)
            hipLaunchKernelGGL(draw_long_perms_kernel, dim3(n_tasks), dim3(kWave), 0, st, tasks, dst, seed, err);
    }
    return hipGetLastError();
}

hipError_t launch_reduce(const ChunkDesc *chunks, int n_chunks, const double *partial, int k,
                         const int32_t *err, double *results, hipStream_t st, int n_groups, int n_surr,
                         double *pv, int32_t *done, int32_t *err_out)
{
    if (n_chunks <= 0)
        return hipSuccess;
    if (pv != nullptr && done == nullptr)
        return hipErrorInvalidValue;
    // the p-values ride on the reduce's last workgroup while the grid is small; above
    // that, every workgroup's device-scope fence and counter atomic cost more than a
    // separate launch (about 1 ms for 16 000 workgroups)
    const int blocks = (n_chunks + 3) / 4;
    const bool fuse = pv != nullptr && blocks <= 256;
    hipLaunchKernelGGL(reduce_kernel, dim3(blocks), dim3(4 * kWave), 0, st, chunks, n_chunks, partial, k, err,
                       results, n_groups, n_surr, fuse ? pv : nullptr, done, err_out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || pv == nullptr || fuse)
        return e;
    hipLaunchKernelGGL(pvalue_kernel, dim3((std::max(n_groups, 1) + 127) / 128), dim3(128), 0, st, results, n_groups,
                       n_surr, pv, err, err_out);
    return hipGetLastError();
}

hipError_t launch_pvalues(const double *results, int n_groups, int n_surr, double *pv, hipStream_t st)
{
    if (n_groups <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(pvalue_kernel, dim3((n_groups + 127) / 128), dim3(128), 0, st, results, n_groups,
                       n_surr, pv, nullptr, nullptr);
    return hipGetLastError();
}

}  // namespace te

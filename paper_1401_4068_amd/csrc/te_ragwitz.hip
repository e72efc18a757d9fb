// te_ragwitz.hip -- the local-predictor score of delay embeddings of the target
// (te_ragwitz): the embedding dimension d and delay tau are chosen as the pair whose
// past state best predicts the next sample with a local predictor (embedding section
// of Wollstadt et al. 2014, after Ragwitz and Kantz).  For each candidate (d, tau) the
// window's points of all trials are pooled; each point's k nearest other points in the
// maximum norm (equal distances ranked by point index) predict its next sample as the
// mean of theirs; the score is the normalised mean squared error.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "te.h"
#include "te_device.h"
#include "te_internal.h"
#include "te_runtime.h"

namespace te {
namespace {

constexpr int kRagMaxDim = TE_RAGWITZ_MAX_DIM;
constexpr int kRagMaxK = TE_RAGWITZ_MAX_K;
constexpr int kScoreThreads = 256;
constexpr int kRagBatch = 16;             // candidates of one launch at most (their tables travel as kernel arguments)
constexpr int kOrderDims = 4;             // state coordinates that order a candidate's points

// One candidate of a launch; offsets in 32-bit words from the workspace's start.
struct RagCand {
    int d, tau, id;
    int64_t rows;                         // states [d][N] in point order
    int64_t copy;                         // states [d][N] in block order
    int64_t box;                          // smallest and largest of each block per coordinate, [2 d][blocks], and its
                                          // smallest point index [blocks]
    int64_t map;                          // order map (order_at)
    int64_t scratch;                      // the ordering's scratch, 64-bit words
};
struct RagArgs {
    int n;
    RagCand c[kRagBatch];
};

// States of the launch's candidates (blockIdx.y): rows[m N + i] = y[r][t - 1 - m tau] for point
// i = r W + (t - w), and with tgt non-null the targets tgt[i] = y[r][t].  A non-finite value sets *bad.
// Also writes the candidate's ordering task.
__global__ void rag_embed_kernel(const float *__restrict__ y, int T, int w, int W, int N, RagArgs a,
                                 float *__restrict__ ws, SortTask *__restrict__ tasks, float *__restrict__ tgt,
                                 int npad, int *__restrict__ bad)
{
    const RagCand c = a.c[blockIdx.y];
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i == 0) {
        SortTask t{};
        t.sig = c.map;
        t.scratch = c.scratch;
        t.key_off = c.rows;
        t.mode = 1;
        t.n = N;
        t.npad = npad;
        t.nd = c.d < kOrderDims ? c.d : kOrderDims;
        tasks[blockIdx.y] = t;
    }
    if (i >= N)
        return;
    const int r = i / W;
    const int t = w + (i - r * W);
    const float *yr = y + (int64_t)r * T;
    bool ok = true;
    for (int m = 0; m < c.d; ++m) {
        const float v = yr[t - 1 - m * c.tau];
        ok = ok && __builtin_isfinite(v);
        ws[c.rows + (int64_t)m * N + i] = v;
    }
    if (tgt != nullptr && blockIdx.y == 0) {
        const float v = yr[t];
        ok = ok && __builtin_isfinite(v);
        tgt[i] = v;
    }
    if (!ok)
        atomicOr(bad, 1);
}

// The states in block order and the blocks' boxes, one wave per block at a time.
__global__ void rag_gather_kernel(RagArgs a, float *__restrict__ ws, int N)
{
    const RagCand c = a.c[blockIdx.y];
    const int32_t *map = reinterpret_cast<const int32_t *>(ws) + c.map;
    const int lane = threadIdx.x & (kWave - 1);
    const int nb = (N + kWave - 1) / kWave;
    for (int qb = (int)(blockIdx.x * blockDim.x) + (int)threadIdx.x - lane; qb < N; qb += (int)(blockDim.x * gridDim.x)) {
        const bool ok = qb + lane < N;
        const int q = ok ? qb + lane : N - 1;
        const int o = min(max(order_at(map, N, q), 0), N - 1);
        const uint32_t least = ~wave_max_u32(~(uint32_t)o);
        if (lane == 0)
            reinterpret_cast<uint32_t *>(ws)[c.box + (int64_t)(2 * c.d) * nb + qb / kWave] = least;
        float x[kRagMaxDim];                              // all loads in flight
#pragma unroll
        for (int m = 0; m < kRagMaxDim; ++m)
            x[m] = m < c.d ? ws[c.rows + (int64_t)m * N + o] : 0.0f;
#pragma unroll
        for (int m = 0; m < kRagMaxDim; ++m)
            if (m < c.d) {
                if (ok)
                    ws[c.copy + (int64_t)m * N + q] = x[m];
                float lo, hi;
                wave_box(x[m], &lo, &hi);
                if (lane == 0) {
                    ws[c.box + (int64_t)(2 * m) * nb + qb / kWave] = lo;
                    ws[c.box + (int64_t)(2 * m + 1) * nb + qb / kWave] = hi;
                }
            }
    }
}

// The KC smallest (distance, index) pairs, ascending: the distance's bits above the index, so that
// one unsigned comparison ranks equal distances by index.  Unfilled places are (inf, 0).
constexpr uint64_t kNone = 0x7f80000000000000ull;
__device__ __forceinline__ uint64_t rank_key(float dist, int index)
{
    return (uint64_t)__builtin_bit_cast(uint32_t, dist) << 32 | (uint32_t)index;
}
template <int KC>
__device__ __forceinline__ void insert_key(uint64_t (&b)[KC], uint64_t x)
{
#pragma unroll
    for (int p = KC - 1; p >= 1; --p)
        b[p] = x < b[p - 1] ? b[p - 1] : (x < b[p] ? x : b[p]);
    b[0] = x < b[0] ? x : b[0];
}
// The k nearest of every point of a block of 64 (block order), the prediction -- the neighbours'
// targets summed in rank order in fp64 -- and its squared error.  W waves of 64 / W references each:
// the block's own points first, every group of 64 / W lanes every W-th of them and the groups' lists
// merged; then, lane = candidate, the blocks whose box the references' current k-th distances
// reach, nearer ones first (a box farther than the k-th distance holds nothing nearer, and nothing
// equally near; rounding is monotone, so the box bound holds for binary32 differences).
// Bound by the latency of a wave's chain of block visits: 175 us for the window of 15 000 points and the
// twelve candidates (d = 1..6, tau = 1, 2; k = 4), all in one launch; every pair of points in index order,
// a launch per candidate, took 2 960 us and merging its segments' lists 1 050 us.
template <int D, int KC, int W>
__device__ __forceinline__ void rag_block(const RagCand &c, const float *ws, const float *tgt, int N, int k,
                                          double *pred, double *sq, float *lds)
{
    constexpr int RPW = kWave / W;             // references per wave
    constexpr int RW = (D + 2 + 3) & ~3;       // LDS row: coordinates, k-th distance, its index
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int nb = (N + kWave - 1) / kWave;
    const int blk = blockIdx.x;
    const float *pts = ws + c.copy;
    const int32_t *map = reinterpret_cast<const int32_t *>(ws) + c.map;
    float *rows = lds + wave * RPW * RW;
    const int i = blk * kWave + wave * RPW + (lane & (RPW - 1));
    const bool valid = i < N && lane < RPW;
    const int ii = min(i, N - 1);
    float ref[D];
#pragma unroll
    for (int m = 0; m < D; ++m)
        ref[m] = pts[(int64_t)m * N + ii];
    uint64_t b[KC];
    // a list longer than k starts with zeros, which nothing displaces: its last entry is the k-th
    const int fill = KC - k;
#pragma unroll
    for (int p = 0; p < KC; ++p)
        b[p] = p < fill ? 0 : kNone;

    // own block (with a ragged last block, the one before it too)
    const int ob0 = (blk > 0 && N - blk * kWave < kWave) ? blk - 1 : blk;
    const int e0 = min(N, (blk + 1) * kWave);
    for (int j0 = ob0 * kWave; j0 < e0; j0 += W) {
        const int j = j0 + lane / RPW, jj = min(j, e0 - 1);
        float dist = absdiff(pts[jj], ref[0]);
#pragma unroll
        for (int m = 1; m < D; ++m)
            dist = fmaxf(dist, absdiff(pts[(int64_t)m * N + jj], ref[m]));
        insert_key<KC>(b, j < e0 && j != i ? rank_key(dist, order_at(map, N, jj)) : kNone);
    }
#pragma unroll
    for (int o = RPW; o < kWave; o <<= 1) {
        uint64_t other[KC];
#pragma unroll
        for (int p = 0; p < KC; ++p)
            other[p] = __shfl_xor((unsigned long long)b[p], o, 64);
#pragma unroll
        for (int p = 0; p < KC; ++p)
            if (p >= fill)
                insert_key<KC>(b, other[p]);
    }
    uint64_t &last = b[KC - 1];
    auto reach = [&]() { return valid ? __builtin_bit_cast(float, (uint32_t)(last >> 32)) : 0.0f; };

    if (lane < RPW) {
#pragma unroll
        for (int m = 0; m < D; ++m)
            rows[lane * RW + m] = ref[m];
        rows[lane * RW + D] = __builtin_bit_cast(float, (uint32_t)(last >> 32));
        rows[lane * RW + D + 1] = __builtin_bit_cast(float, (uint32_t)last);
    }
    __builtin_amdgcn_wave_barrier();

    // the box of the wave's own references
    const float *bx = ws + c.box;
    float blo[D], bhi[D];
#pragma unroll
    for (int m = 0; m < D; ++m) {
        float lo = ref[m] != ref[m] ? -kInf : ref[m], hi = ref[m] != ref[m] ? kInf : ref[m];
#pragma unroll
        for (int o = 1; o < RPW; o <<= 1) {
            lo = fminf(lo, __shfl_xor(lo, o, 64));
            hi = fmaxf(hi, __shfl_xor(hi, o, 64));
        }
        blo[m] = readlane_f(lo, 0);
        bhi[m] = readlane_f(hi, 0);
    }
    float lim = -kInf;
    for (int sw = 0; sw < 4 && nb > 1; ++sw) {
        float cm = wave_max(reach());
        const float share = sw == 0 ? 0.05f : (sw == 1 ? 0.15f : 0.4f);
        const float nlim = sw == 3 ? kInf : fmaxf(lim, share * cm);
        if (nlim == lim)
            continue;
        for (int b0 = 0; b0 < nb; b0 += kWave) {
            const int bb = min(b0 + lane, nb - 1);
            float lo[D], hi[D], g = -kInf;
#pragma unroll
            for (int m = 0; m < D; ++m) {
                lo[m] = bx[(int64_t)(2 * m) * nb + bb];
                hi[m] = bx[(int64_t)(2 * m + 1) * nb + bb];
                g = fmaxf(g, fmaxf(lo[m] - bhi[m], blo[m] - hi[m]));
            }
            const int bl = b0 + lane;
            uint64_t want = ballot(bl < nb && (bl < ob0 || bl > blk) && g >= lim && (g < nlim || sw == 3) && !(g > cm));
            if (want == 0)
                continue;
            if ((want & ballot(g == cm)) != 0) {
                // boxes at the largest k-th distance itself: their points' indices decide
                const uint32_t worst = wave_max_u32(valid && reach() == cm ? (uint32_t)last : 0u);
                const uint32_t least = reinterpret_cast<const uint32_t *>(bx)[(int64_t)(2 * D) * nb + bb];
                want &= ~ballot(g == cm && least >= worst);
                if (want == 0)
                    continue;
            }
            do {
                const int cc = __builtin_ctzll(want);
                want = clear_bit(want, cc);
                float far = -kInf;                        // of the lane's reference from the block's box
#pragma unroll
                for (int m = 0; m < D; ++m)
                    far = fmaxf(far, fmaxf(readlane_f(lo[m], cc) - ref[m], ref[m] - readlane_f(hi[m], cc)));
                uint64_t todo = ballot(valid && !(far > reach()));
                if (todo == 0)
                    continue;
                const int idx = (b0 + cc) * kWave + lane;
                const int jj = min(idx, N - 1);
                float cand[D];
#pragma unroll
                for (int m = 0; m < D; ++m)
                    cand[m] = pts[(int64_t)m * N + jj];
                cand[0] = idx < N ? cand[0] : kInf;
                const int ci = order_at(map, N, jj);
                do {
                    const int r = __builtin_ctzll(todo);
                    todo = clear_bit(todo, r);
                    float rr[RW];
#pragma unroll
                    for (int x = 0; x < RW / 4; ++x) {
                        const f4v q4 = reinterpret_cast<const f4v *>(rows + r * RW)[x];
                        rr[4 * x + 0] = q4.x;
                        rr[4 * x + 1] = q4.y;
                        rr[4 * x + 2] = q4.z;
                        rr[4 * x + 3] = q4.w;
                    }
                    float dist = absdiff(rr[0], cand[0]);
#pragma unroll
                    for (int m = 1; m < D; ++m)
                        dist = fmaxf(dist, absdiff(rr[m], cand[m]));
                    if (ballot(dist <= rr[D]) == 0)
                        continue;
                    keep_branch();
                    const uint64_t key = rank_key(dist, ci);
                    uint64_t bar = (uint64_t)__builtin_bit_cast(uint32_t, rr[D]) << 32 |
                                   __builtin_bit_cast(uint32_t, rr[D + 1]);
                    uint64_t hit = ballot(dist <= rr[D] && key < bar);   // a distance that is no number hits nothing
                    if (hit == 0)
                        continue;
                    do {
                        const int x = __builtin_ctzll(hit);
                        hit = clear_bit(hit, x);
                        const uint64_t kx =
                            (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(key >> 32), x) << 32 |
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, x);
                        if (lane == r)
                            insert_key<KC>(b, kx);
                        bar = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(last >> 32), r) << 32 |
                              (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)last, r);
                        hit &= ballot(key < bar);
                    } while (hit != 0);
                    if (lane == r) {
                        rows[r * RW + D] = __builtin_bit_cast(float, (uint32_t)(last >> 32));
                        rows[r * RW + D + 1] = __builtin_bit_cast(float, (uint32_t)last);
                    }
                    __builtin_amdgcn_wave_barrier();
                } while (todo != 0);
            } while (want != 0);
            cm = wave_max(reach());
        }
        lim = nlim;
    }
    if (!valid)
        return;
    double s = 0.0;
#pragma unroll
    for (int p = 0; p < KC; ++p)
        if (p >= fill)
            s += (double)tgt[min((uint32_t)b[p], (uint32_t)(N - 1))];
    const double yhat = s / (double)k;
    const int o = min(max(order_at(map, N, i), 0), N - 1);
    if (pred != nullptr)
        pred[o] = yhat;
    const double e = (double)tgt[o] - yhat;
    sq[o] = e * e;
}

template <int KC, int W>
__global__ void __launch_bounds__(W * kWave) rag_search_kernel(RagArgs a, const float *__restrict__ ws,
                                                               const float *__restrict__ tgt, int N, int k,
                                                               double *pred, double *sq)
{
    __shared__ __attribute__((aligned(16))) float lds[kWave * ((kRagMaxDim + 2 + 3) & ~3)];
    const RagCand c = a.c[blockIdx.y];
    double *p = pred != nullptr ? pred + (int64_t)c.id * N : nullptr;
    double *q = sq + (int64_t)c.id * N;
    switch (c.d) {
    case 1: rag_block<1, KC, W>(c, ws, tgt, N, k, p, q, lds); break;
    case 2: rag_block<2, KC, W>(c, ws, tgt, N, k, p, q, lds); break;
    case 3: rag_block<3, KC, W>(c, ws, tgt, N, k, p, q, lds); break;
    case 4: rag_block<4, KC, W>(c, ws, tgt, N, k, p, q, lds); break;
    case 5: rag_block<5, KC, W>(c, ws, tgt, N, k, p, q, lds); break;
    case 6: rag_block<6, KC, W>(c, ws, tgt, N, k, p, q, lds); break;
    case 7: rag_block<7, KC, W>(c, ws, tgt, N, k, p, q, lds); break;
    default: rag_block<8, KC, W>(c, ws, tgt, N, k, p, q, lds); break;
    }
}

// Few points: no order, every pair.  A wave takes R references and has its lanes take every 64th point
// each, a list of the k nearest of them per lane; the k-th smallest of the lanes' nearest distances bounds
// the reference's k-th, so that after a few rounds hardly a point is inserted.  The lists are merged by
// taking their smallest entry k times, and prediction and error are formed as above.
// Bound by issue: one candidate of d = 8, 15 000 points, k = 4: 239 us a call, 342 in block order.
constexpr int kFewWaves = 4;

template <int D, int KC, int R>
__device__ __forceinline__ void rag_few(const RagCand &c, const float *ws, const float *tgt, int N, int k, double *pred,
                                        double *sq)
{
    constexpr int U = D <= 4 ? 4 : 2;          // rounds whose loads are in flight together
    const int lane = threadIdx.x & (kWave - 1);
    const int i0 = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kFewWaves + threadIdx.x / kWave) * R);
    if (i0 >= N)
        return;
    const float *rows = ws + c.rows;
    float ref[R][D], bound[R];
    uint64_t b[R][KC];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        bound[r] = kInf;
#pragma unroll
        for (int m = 0; m < D; ++m)
            ref[r][m] = uload(rows + (int64_t)m * N + min(i0 + r, N - 1));
#pragma unroll
        for (int p = 0; p < KC; ++p)
            b[r][p] = kNone;
    }
    int next = 2;                              // rounds after which the bounds are taken again
    for (int j0 = 0, round = 0; j0 < N; j0 += U * kWave) {
        float x[U][D];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int m = 0; m < D; ++m)
                x[u][m] = vload_at(rows + (int64_t)m * N, (uint32_t)min(j0 + u * kWave + lane, N - 1) * 4u);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * kWave + lane;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float dist = absdiff(x[u][0], ref[r][0]);
#pragma unroll
                for (int m = 1; m < D; ++m)
                    dist = fmaxf(dist, absdiff(x[u][m], ref[r][m]));
                const bool in = j < N && j != i0 + r && dist < bound[r];
                if (ballot(in)) {
                    keep_branch();
                    insert_key<KC>(b[r], in ? rank_key(dist, j) : kNone);
                }
            }
        }
        round += U;
        if (round >= next && j0 + U * kWave < N) {
            next = 2 * round;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                uint32_t h = (uint32_t)(b[r][0] >> 32), v;
                int left = k;
                do {
                    v = ~wave_max_u32(~h);
                    left -= __builtin_popcountll(ballot(h == v));
                    h = h == v ? ~0u : h;
                } while (left > 0);
                bound[r] = __builtin_bit_cast(float, v);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int near = 0;                          // lane p: the p-th nearest
        for (int p = 0; p < k; ++p) {
            const uint32_t hi = (uint32_t)(b[r][0] >> 32), lo = (uint32_t)b[r][0];
            const uint32_t v = ~wave_max_u32(~hi);
            const uint32_t l = ~wave_max_u32(hi == v ? ~lo : 0u);
            if (hi == v && lo == l) {
#pragma unroll
                for (int q = 0; q + 1 < KC; ++q)
                    b[r][q] = b[r][q + 1];
                b[r][KC - 1] = kNone;
            }
            near = lane == p ? (int)l : near;
        }
        const float t = tgt[min((uint32_t)near, (uint32_t)(N - 1))];
        double s = 0.0;
        for (int p = 0; p < k; ++p)
            s += (double)readlane_f(t, p);
        const int i = i0 + r;
        if (lane == 0 && i < N) {
            const double yhat = s / (double)k;
            if (pred != nullptr)
                pred[i] = yhat;
            const double e = (double)tgt[i] - yhat;
            sq[i] = e * e;
        }
    }
}

template <int KC, int R>
__global__ void __launch_bounds__(kFewWaves * kWave) rag_few_kernel(RagArgs a, const float *__restrict__ ws,
                                                                    const float *__restrict__ tgt, int N, int k,
                                                                    double *pred, double *sq)
{
    const RagCand c = a.c[blockIdx.y];
    double *p = pred != nullptr ? pred + (int64_t)c.id * N : nullptr;
    double *q = sq + (int64_t)c.id * N;
    switch (c.d) {
    case 1: rag_few<1, KC, R>(c, ws, tgt, N, k, p, q); break;
    case 2: rag_few<2, KC, R>(c, ws, tgt, N, k, p, q); break;
    case 3: rag_few<3, KC, R>(c, ws, tgt, N, k, p, q); break;
    case 4: rag_few<4, KC, R>(c, ws, tgt, N, k, p, q); break;
    case 5: rag_few<5, KC, R>(c, ws, tgt, N, k, p, q); break;
    case 6: rag_few<6, KC, R>(c, ws, tgt, N, k, p, q); break;
    case 7: rag_few<7, KC, R>(c, ws, tgt, N, k, p, q); break;
    default: rag_few<8, KC, R>(c, ws, tgt, N, k, p, q); break;
    }
}

template <int KC>
void launch_rag_search(const RagArgs &a, const float *ws, const float *tgt, int N, int k, double *pred, double *sq, int w,
                       hipStream_t st)
{
    const dim3 grid((unsigned)((N + kWave - 1) / kWave), (unsigned)a.n), block(w * kWave);
    if (w == 8)
        rag_search_kernel<KC, 8><<<grid, block, 0, st>>>(a, ws, tgt, N, k, pred, sq);
    else
        rag_search_kernel<KC, 4><<<grid, block, 0, st>>>(a, ws, tgt, N, k, pred, sq);
}

// (the list capacity is the smallest of 4, 8, 16 that holds k)
hipError_t launch_rag_search(const RagArgs &a, const float *ws, const float *tgt, int N, int k, double *pred, double *sq,
                             hipStream_t st)
{
    // blocks of the launch to eight waves each while those are few for the chip (us a call, eight / four
    // waves: 705 blocks (15 000 points, d = 2, 4, 6, k = 4) 263 / 287, 1 880 (d = 1..8) 428 / 417 and at k = 8
    // 556 / 578, 2 820 (d = 1..6, two delays) 365 / 362 and 511 / 497)
    const int w = (int64_t)((N + kWave - 1) / kWave) * a.n <= 2048 ? 8 : 4;
    if (k <= 4)
        launch_rag_search<4>(a, ws, tgt, N, k, pred, sq, w, st);
    else if (k <= 8)
        launch_rag_search<8>(a, ws, tgt, N, k, pred, sq, w, st);
    else
        launch_rag_search<16>(a, ws, tgt, N, k, pred, sq, w, st);
    return hipGetLastError();
}

// Launches of at most so many pairs of points go without an order.  us a call, k = 4, every pair / ordered
// (AR series, values rounded to integers): 4 000 points, 12 candidates (192 M pairs) 175 / 200 and 147 / 226;
// 24 candidates (256 + 128 M) 338 / 378 and 281 / 418; 15 000 points, one of d = 8 (225 M) 239 / 342 and
// 224 / 429, one of d = 3 183 / 178 and 156 / 185; d = 2, 4, 6 (675 M) 382 / 263 and 327 / 301.
constexpr int64_t kFewPairs = 1 << 28;

template <int KC>
void launch_rag_few(const RagArgs &a, const float *ws, const float *tgt, int N, int k, double *pred, double *sq,
                    hipStream_t st)
{
    // two references to a wave share the points' loads; one while the waves are few (us a call, one / two:
    // 4 000 points, k = 16, one candidate 115 / 127, 12 candidates 514 / 508)
    const int r = (int64_t)N * a.n <= 8192 ? 1 : 2;
    const dim3 grid((unsigned)((N + kFewWaves * r - 1) / (kFewWaves * r)), (unsigned)a.n), block(kFewWaves * kWave);
    if (r == 1)
        rag_few_kernel<KC, 1><<<grid, block, 0, st>>>(a, ws, tgt, N, k, pred, sq);
    else
        rag_few_kernel<KC, 2><<<grid, block, 0, st>>>(a, ws, tgt, N, k, pred, sq);
}

hipError_t launch_rag_few(const RagArgs &a, const float *ws, const float *tgt, int N, int k, double *pred, double *sq,
                          hipStream_t st)
{
    if (k <= 4)
        launch_rag_few<4>(a, ws, tgt, N, k, pred, sq, st);
    else if (k <= 8)
        launch_rag_few<8>(a, ws, tgt, N, k, pred, sq, st);
    else
        launch_rag_few<16>(a, ws, tgt, N, k, pred, sq, st);
    return hipGetLastError();
}

// Fixed-order sum over a workgroup of kScoreThreads threads.
__device__ double block_sum(double v, double *part)
{
    const int tid = (int)threadIdx.x;
    part[tid] = v;
    __syncthreads();
    for (int s = kScoreThreads / 2; s > 0; s >>= 1) {
        if (tid < s)
            part[tid] += part[tid + s];
        __syncthreads();
    }
    const double r = part[0];
    __syncthreads();
    return r;
}

// Score of candidate c = blockIdx.x: sum of squared errors / sum of squared deviations
// of the targets from their mean (NaN if the targets are constant).  One workgroup a candidate keeps the
// order of the sums; bound by the latency of its loads, eight at a time (15 000 points: 11 us, one at a
// time 25 us).
__global__ void __launch_bounds__(kScoreThreads) rag_score_kernel(const float *__restrict__ tgt,
                                                                   const double *__restrict__ sq, int N,
                                                                   double *__restrict__ score)
{
    __shared__ double part[kScoreThreads];
    const int c = (int)blockIdx.x;
    constexpr int U = 8;                                  // loads in flight per thread
    double a = 0.0;
    for (int i0 = (int)threadIdx.x; i0 < N; i0 += U * kScoreThreads) {
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            x[u] = tgt[min(i0 + u * kScoreThreads, N - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kScoreThreads < N)
                a += (double)x[u];
    }
    const double mean = block_sum(a, part) / (double)N;
    double v = 0.0, e = 0.0;
    for (int i0 = (int)threadIdx.x; i0 < N; i0 += U * kScoreThreads) {
        float x[U];
        double q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + u * kScoreThreads, N - 1);
            x[u] = tgt[i];
            q[u] = sq[(int64_t)c * N + i];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kScoreThreads < N) {
                const double dlt = (double)x[u] - mean;
                v += dlt * dlt;
                e += q[u];
            }
    }
    const double V = block_sum(v, part);
    const double E = block_sum(e, part);
    if (threadIdx.x == 0)
        score[c] = V > 0.0 ? E / V : __builtin_nan("");
}

// Words of one candidate's part of the search area: states in block order, boxes, order map, and the
// ordering's scratch (codes, or the keys of spaces that are sorted whole) above kSortLds points.
struct RagPart {
    int64_t box, map, scratch, total;
};

RagPart rag_part(int64_t N, int d)
{
    auto up = [](int64_t v) { return (v + 15) / 16 * 16; };
    RagPart p;
    p.box = up(N * d);
    p.map = p.box + up((2 * d + 1) * ((N + kWave - 1) / kWave));
    p.scratch = p.map + up(N);
    int64_t words = 0;
    if (N > kSortLds)
        words = sorted_whole((int)N) ? 2 * (int64_t)sort_npad((int)N) : (N + 1) / 2;
    p.total = p.scratch + up(words);
    return p;
}

// 128 bytes a point of the search area for each of these runs of at least 64 points: the size callers have
// reserved for it, of which a candidate's part takes at most 56 bytes a point and 320 bytes.
int64_t rag_runs(int64_t N)
{
    auto runs = [N](int64_t refs) {
        const int64_t groups = (N + refs - 1) / refs;
        const int64_t want = std::min<int64_t>(64, std::max<int64_t>(1, (16384 + groups - 1) / groups));
        const int64_t len = std::max<int64_t>(64, ((N + want - 1) / want + 7) / 8 * 8);
        return (N + len - 1) / len;
    };
    return std::max(runs(kWave), runs(4 * kWave));
}

// Workspace layout: flag | targets [N] | states of each candidate [d_c][N] | squared errors [n_cand][N] |
// scores [n_cand] | search area (ordering tasks, then parts of as many candidates at a time as fit); each
// part 256-byte aligned.
struct RagLayout {
    size_t tgt = 0, sq = 0, score = 0, area = 0, total = 0;
    std::vector<size_t> rows;
};

RagLayout rag_layout(int64_t N, const int32_t *dims, int n_cand)
{
    RagLayout L;
    size_t o = 256;
    L.tgt = o;
    o += align_up(sizeof(float) * (size_t)N, 256);
    for (int c = 0; c < n_cand; ++c) {
        L.rows.push_back(o);
        o += align_up(sizeof(float) * (size_t)N * (size_t)dims[c], 256);
    }
    L.sq = o;
    o += align_up(sizeof(double) * (size_t)N * (size_t)n_cand, 256);
    L.score = o;
    o += align_up(sizeof(double) * (size_t)n_cand, 256);
    const int64_t lists = rag_runs(N) * kRagMaxK * N;
    L.area = o;
    o += 2 * align_up(sizeof(float) * (size_t)lists, 256);
    L.total = o;
    return L;
}

te_status rag_check(int32_t n_trials, int32_t n_samples, int32_t window_start, int32_t window_len,
                    const int32_t *dims, const int32_t *taus, int32_t n_cand, int32_t k)
{
    if (!dims || !taus)
        return fail(TE_ERR_INVALID, "null argument");
    if (n_cand < 1 || n_cand > TE_RAGWITZ_MAX_CANDIDATES)
        return fail(TE_ERR_INVALID, "n_cand must be in 1..%d", TE_RAGWITZ_MAX_CANDIDATES);
    if (k < 1 || k > kRagMaxK)
        return fail(TE_ERR_INVALID, "k must be in 1..%d", kRagMaxK);
    if (n_trials < 1 || window_len < 1)
        return fail(TE_ERR_INVALID, "n_trials and window_len must be >= 1");
    if (window_start < 0 || (int64_t)window_start + window_len > n_samples)
        return fail(TE_ERR_INVALID, "window [%d, %d) runs past n_samples = %d", window_start,
                    window_start + window_len, n_samples);
    const int64_t N = (int64_t)n_trials * window_len;
    if (N <= k || N > kMaxWindowPoints)
        return fail(TE_ERR_INVALID, "the window pools %lld points; need k < N <= %d", (long long)N,
                    kMaxWindowPoints);
    for (int c = 0; c < n_cand; ++c) {
        if (dims[c] < 1 || dims[c] > kRagMaxDim || taus[c] < 1)
            return fail(TE_ERR_INVALID, "candidate %d: d = %d, tau = %d (need 1 <= d <= %d, tau >= 1)", c, dims[c],
                        taus[c], kRagMaxDim);
        if ((int64_t)window_start < 1 + (int64_t)(dims[c] - 1) * taus[c])
            return fail(TE_ERR_INVALID, "candidate %d: the window starts at %d but the state needs %lld samples of "
                        "history", c, window_start, (long long)(1 + (int64_t)(dims[c] - 1) * taus[c]));
    }
    return TE_OK;
}

}  // namespace
}  // namespace te

using namespace te;

extern "C" {

te_status te_ragwitz_workspace_bytes(int32_t n_trials, int32_t window_len, const int32_t *dims, int32_t n_cand,
                                     size_t *bytes)
{
    clear_error();
    if (!dims || !bytes)
        return fail(TE_ERR_INVALID, "null argument");
    if (n_trials < 1 || window_len < 1 || n_cand < 1 || n_cand > TE_RAGWITZ_MAX_CANDIDATES)
        return fail(TE_ERR_INVALID, "bad geometry");
    for (int c = 0; c < n_cand; ++c)
        if (dims[c] < 1 || dims[c] > kRagMaxDim)
            return fail(TE_ERR_INVALID, "candidate %d: d = %d outside 1..%d", c, dims[c], kRagMaxDim);
    *bytes = rag_layout((int64_t)n_trials * window_len, dims, n_cand).total;
    return TE_OK;
}

te_status te_ragwitz(const float *y, int32_t n_trials, int32_t n_samples, int32_t window_start, int32_t window_len,
                     const int32_t *dims, const int32_t *taus, int32_t n_cand, int32_t k, void *ws_, size_t ws_bytes,
                     void *hip_stream, double *pred, double *score)
{
    TraceRange trace_range("te.ragwitz");
    clear_error();
    if (!y || !ws_ || !score)
        return fail(TE_ERR_INVALID, "null argument");
    te_status s = rag_check(n_trials, n_samples, window_start, window_len, dims, taus, n_cand, k);
    if (s != TE_OK)
        return s;
    const int N = n_trials * window_len;
    const RagLayout L = rag_layout(N, dims, n_cand);
    if (ws_bytes < L.total)
        return fail(TE_ERR_NOMEM, "workspace %zu bytes < %zu", ws_bytes, L.total);
    char *ws = static_cast<char *>(ws_);
    hipStream_t st = (hipStream_t)hip_stream;
    int *bad = reinterpret_cast<int *>(ws);
    float *tgt = reinterpret_cast<float *>(ws + L.tgt);
    double *sq = reinterpret_cast<double *>(ws + L.sq);
    double *dscore = reinterpret_cast<double *>(ws + L.score);
    hipError_t e = launch_fill_i32(bad, 0, 1, st);
    if (e != hipSuccess)
        return hip_fail(e, "fill");
    float *wsf = reinterpret_cast<float *>(ws);
    const int64_t area_words = (int64_t)((L.total - L.area) / sizeof(float));
    const int npad = sort_npad(N);
    for (int c0 = 0; c0 < n_cand;) {
        // as many candidates as the search area holds
        RagArgs a{};
        int64_t words = 0;
        const int64_t area = (int64_t)(L.area / sizeof(float));
        auto task_words = [](int n) { return ((int64_t)n * (int64_t)sizeof(SortTask) / 4 + 15) / 16 * 16; };
        while (a.n < kRagBatch && c0 + a.n < n_cand) {
            const RagPart p = rag_part(N, dims[c0 + a.n]);
            if (a.n > 0 && task_words(a.n + 1) + words + p.total > area_words)
                break;
            words += p.total;
            ++a.n;
        }
        int64_t o = area + task_words(a.n);
        for (int c = 0; c < a.n; ++c) {
            const RagPart p = rag_part(N, dims[c0 + c]);
            a.c[c] = RagCand{dims[c0 + c], taus[c0 + c], c0 + c, (int64_t)(L.rows[c0 + c] / sizeof(float)), o,
                             o + p.box, o + p.map, (o + p.scratch) / 2};
            o += p.total;
        }
        if (o > area + area_words)
            return fail(TE_ERR_NOMEM, "the search area does not hold a candidate's part");
        SortTask *tasks = reinterpret_cast<SortTask *>(wsf + area);
        rag_embed_kernel<<<dim3((unsigned)((N + 255) / 256), (unsigned)a.n), dim3(256), 0, st>>>(
            y, n_samples, window_start, window_len, N, a, wsf, tasks, c0 == 0 ? tgt : nullptr, npad, bad);
        if ((e = hipGetLastError()) != hipSuccess)
            return hip_fail(e, "rag_embed_kernel");
        if ((int64_t)N * N * a.n <= kFewPairs) {
            if ((e = launch_rag_few(a, wsf, tgt, N, k, pred, sq, st)) != hipSuccess)
                return hip_fail(e, "rag_few_kernel");
            c0 += a.n;
            continue;
        }
        SortSizes sizes;
        for (int c = 0; c < a.n; ++c)
            sizes.add(N);
        if ((e = launch_sort(nullptr, wsf, N, tasks, sizes, reinterpret_cast<int32_t *>(ws),
                             reinterpret_cast<uint64_t *>(ws), 0, 0, 0, 0, st)) != hipSuccess)
            return hip_fail(e, "ordering");
        const dim3 gather((unsigned)std::min(1024, (N + 255) / 256), (unsigned)a.n);   // a wave per block of points
        rag_gather_kernel<<<gather, dim3(256), 0, st>>>(a, wsf, N);
        if ((e = hipGetLastError()) != hipSuccess)
            return hip_fail(e, "rag_gather_kernel");
        if ((e = launch_rag_search(a, wsf, tgt, N, k, pred, sq, st)) != hipSuccess)
            return hip_fail(e, "rag_search_kernel");
        c0 += a.n;
    }
    rag_score_kernel<<<dim3((unsigned)n_cand), dim3(kScoreThreads), 0, st>>>(tgt, sq, N, dscore);
    if ((e = hipGetLastError()) != hipSuccess)
        return hip_fail(e, "rag_score_kernel");
    int bad_h = 0;
    std::vector<double> sc(n_cand);
    if ((e = hipMemcpyAsync(&bad_h, bad, sizeof(int), hipMemcpyDeviceToHost, st)) != hipSuccess ||
        (e = hipMemcpyAsync(sc.data(), dscore, sizeof(double) * n_cand, hipMemcpyDeviceToHost, st)) != hipSuccess)
        return hip_fail(e, "hipMemcpyAsync");
    {
        TraceRange wait_range("te.wait");
        if ((e = hipStreamSynchronize(st)) != hipSuccess)
            return hip_fail(e, "hipStreamSynchronize");
    }
    if (bad_h)
        return fail(TE_ERR_INVALID, "non-finite value in the window or its history");
    for (int c = 0; c < n_cand; ++c)
        score[c] = sc[c];
    return TE_OK;
}

}  // extern "C"

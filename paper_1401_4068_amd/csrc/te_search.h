// te_search.h -- the KSG searches over ordered search spaces (text before eq. 9).
//
// A search space (chunk, eq. 10) is stored in an order in which 64 consecutive
// points -- a block -- lie close together in the target past (order_kernel), with
// the bounding box of every block over the target-past coordinates (embed_kernel).
// All three marginal balls of eq. 8, and the joint ball, lie inside the target-past
// ball of the same radius, so a block whose box is at least a point's radius away
// holds nothing that any of its searches could use: fl32(lo - r) and fl32(r - hi)
// bound fl32(|c - r|) of every c in [lo, hi] from below, rounding being monotone.
// Both passes are therefore exact and see a few per cent of a large chunk
// (49 400 points, d_y = 3: 4.8 % of its pairs per pass, against 23 % when the chunk
// was sorted by its first target-past coordinate alone and cut to a window of it).
//
// The chunks of one window (its original and its surrogates, or its delays) share
// the (y_t', Y_past) block, its order and its boxes and differ only in the source
// block; up to V of them are searched per work item: the target differences of a
// pair are taken once, and only the source part is evaluated per chunk.  With
//   d_TP = max(d_T, d_P),  d_J(v) = max(d_TP, d_S(v)),
// n_P counts [d_P < eps_v], n_TP [d_TP < eps_v], n_PS [max(d_P, d_S(v)) < eps_v].
// Radii, counts and per-item sums do not depend on V: the same float operations
// decide every comparison, and a block's terms are summed in the same lanes.
//
// A work item is one set of chunks and one block of 64 references.  Large launches are
// persistent: every wavefront pulls items from the queue of its XCD until all queues are
// empty.  Small ones give every block a workgroup of W waves, 64 / W references to each
// (waves_to_a_block).

#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "te_device.h"
#include "te_internal.h"

namespace te {

namespace {

// A block that at least this many of the 64 references reach is searched with
// lane = reference (its insertions run in all lanes at once); below that with
// lane = candidate against the references that reach it only.
constexpr int kDense = 44;
// Work item -> chunk run: a set is a run of consecutive chunk descriptors
// [set_first[c], set_first[c+1]) (single chunks without set_first); its first
// descriptor supplies tp, box, n, item0 and block0, each descriptor its own s and
// pbase.  Sets with fewer than V chunks repeat their last chunk in the unused
// variant slots and do not store those slots' sums.
template <int DY, int DX, int V, int KP1, bool GENERIC, int SLOTS, bool OUT, int W>
__device__ __forceinline__ void block_search(const SearchArgs &a)
{
    constexpr int DT = 1 + DY;                 // shared coordinates: y_t' and the target past
    constexpr int NR = DT + V * DX + V;        // LDS row: shared coordinates, V source blocks, V radii
    constexpr int RW = (NR + 3) & ~3;
    constexpr int MO = DT > DX ? DT : DX;      // coordinate offsets shared by the target and source blocks
    extern __shared__ __attribute__((aligned(16))) float rows[];   // waves per workgroup x 64 x RW floats
    __shared__ double wsum[V][W > 0 ? W : 1];
    const int lane = threadIdx.x & (kWave - 1);
    const int k = GENERIC ? a.k : KP1 - 1;
    constexpr int RPW = W > 0 ? kWave / W : kWave;   // references per wave
    float *prow = rows + (threadIdx.x / kWave) * (kWave * RW);

    const int nq = a.n_parts > 1 ? a.n_parts : 1;
    int qp = (int)(blockIdx.x % (unsigned)nq);   // this wave's queue
    int drained = 0;                              // queues found empty so far
    int last_ci = 0, last_lo = 0, last_hi = 0;    // the previous item's set and its item range
    unsigned long long work1 = 0, work2 = 0, shared1 = 0, shared2 = 0;
    for (;;) {
        // ---- claim the next work item (wave-uniform)
        int q = (int)blockIdx.x;
        if (W == 0) {
            if (lane == 0)
                q = atomicAdd(a.counter + qp, 1);
            q = __builtin_amdgcn_readlane(q, 0);
        }
        if (W == 0 && nq > 1) {
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
        // consecutive items of a queue are mostly blocks of one set
        if (q < last_lo || q >= last_hi) {
            last_ci = find_chunk(a.item_start, a.n_chunks, q);
            last_lo = uload_i(a.item_start + last_ci);
            last_hi = last_ci + 1 < a.n_chunks ? uload_i(a.item_start + last_ci + 1) : a.n_items;
        }
        int c0 = last_ci, cnt = 1;                 // first chunk and number of chunks of the set
        if (V > 1) {
            c0 = uload_i(a.set_first + last_ci);
            cnt = uload_i(a.set_first + last_ci + 1) - c0;
        }
        const char *w0 = reinterpret_cast<const char *>(a.chunks + c0);
        const float *tb = a.base + uload_l(reinterpret_cast<const int64_t *>(w0 + offsetof(ChunkDesc, tp)));
        const float *bx = a.base + uload_l(reinterpret_cast<const int64_t *>(w0 + offsetof(ChunkDesc, geo)));
        const int n = uload_i(reinterpret_cast<const int32_t *>(w0 + offsetof(ChunkDesc, n)));
        const int item0 = uload_i(reinterpret_cast<const int32_t *>(w0 + offsetof(ChunkDesc, item0)));
        const int block0 = uload_i(reinterpret_cast<const int32_t *>(w0 + offsetof(ChunkDesc, block0)));
        const float *sb[V];                            // source block of each variant
        int64_t pb[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const char *wv = reinterpret_cast<const char *>(a.chunks + c0 + min(v, cnt - 1));
            sb[v] = a.base + uload_l(reinterpret_cast<const int64_t *>(wv + offsetof(ChunkDesc, s)));
            pb[v] = uload_l(reinterpret_cast<const int64_t *>(wv + offsetof(ChunkDesc, pbase)));
        }
        // Coordinate m of a block: sets address it by a 32-bit byte offset from the block's start,
        // shared by their blocks (a window holds at most kMaxWindowPoints points); a single chunk,
        // which may be larger, by row pointers.
        uint32_t moff[MO];
#pragma unroll
        for (int m = 0; m < MO; ++m)
            moff[m] = V > 1 ? (uint32_t)((int64_t)m * n * 4) : 0u;
        auto row = [&](const float *p, int m) { return V > 1 ? p : p + (int64_t)m * n; };
        const int blk = q - item0 + block0;
        const int nb = (n + kWave - 1) / kWave;
        const int r0 = blk * kWave + (W > 0 ? (int)(threadIdx.x / kWave) * RPW : 0);

        // ---- pass 1
        // (with W waves to a block, every RPW lanes hold the wave's references again, the first ones in use)
        const int i = r0 + (lane & (RPW - 1));
        const bool valid = i < n && lane < RPW;
        const int ii = min(i, n - 1);
        float rt[DT];
        float rs[V][DX];
#pragma unroll
        for (int m = 0; m < DT; ++m)
            rt[m] = vload_at(row(tb, m), moff[m] + (uint32_t)ii * 4u);
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int m = 0; m < DX; ++m)
                rs[v][m] = vload_at(row(sb[v], m), moff[m] + (uint32_t)ii * 4u);
        // The k+1 smallest joint distances of the lane's reference per variant, itself
        // included (distance 0): the radius is the (k+1)-th, the k-th neighbour without self.
        // A list longer than that starts with zeros, which nothing displaces, so the radius is
        // always its last entry.
        const int fill = GENERIC ? KP1 - 1 - k : 0;
        float best[V][KP1];
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int s = 0; s < KP1; ++s)
                best[v][s] = s < fill ? 0.0f : kInf;
        auto cur = [&](int v) { return best[v][KP1 - 1]; };
        auto insert = [&](int v, float x) { insert_sorted<KP1>(best[v], x); };
        // largest current radius over the variants (0 in lanes past the chunk's end): a
        // candidate at least that far away is of no use to any variant
        auto curmax = [&]() {
            float c = cur(0);
#pragma unroll
            for (int v = 1; v < V; ++v)
                c = fmaxf(c, cur(v));
            return valid ? c : 0.0f;
        };

        // LDS row of a reference: its coordinates, then its current radius per variant
        auto store_row = [&](const float (&ct)[DT], const float (&cs)[V][DX]) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int m = 0; m < DT; ++m)
                prow[lane * RW + m] = ct[m];
#pragma unroll
            for (int v = 0; v < V; ++v) {
#pragma unroll
                for (int m = 0; m < DX; ++m)
                    prow[lane * RW + DT + v * DX + m] = cs[v][m];
                prow[lane * RW + DT + V * DX + v] = cur(v);
            }
            __builtin_amdgcn_wave_barrier();
        };
        auto read_row = [&](int r, float (&rr)[RW]) {
            const f4v *rowv = reinterpret_cast<const f4v *>(prow + r * RW);
#pragma unroll
            for (int x = 0; x < RW / 4; ++x) {
                const f4v q4 = rowv[x];
                rr[4 * x + 0] = q4.x;
                rr[4 * x + 1] = q4.y;
                rr[4 * x + 2] = q4.z;
                rr[4 * x + 3] = q4.w;
            }
        };
        auto store_radii = [&]() {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int v = 0; v < V; ++v)
                prow[lane * RW + DT + V * DX + v] = cur(v);
            __builtin_amdgcn_wave_barrier();
        };
        // Block b's candidates, one per lane; past the chunk's end the last point moved to +inf, outside
        // every ball: in all coordinates where a reference may be infinite itself (pre-embedded points),
        // else in one.  (Added, not selected: back to back, selects on VCC issue one in 23 clocks.)
        auto load_block = [&](int b, float (&ct)[DT], float (&cs)[V][DX]) {
            const int idx = b * kWave + lane;
            const bool ok = idx < n;
            const uint32_t ic4 = (uint32_t)(ok ? idx : n - 1) * 4u;
            const float away = ok ? 0.0f : kInf;
#pragma unroll
            for (int m = 0; m < DT; ++m) {
                const float x = vload_at(row(tb, m), moff[m] + ic4);
                ct[m] = OUT || m == 1 ? x + away : x;
            }
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int m = 0; m < DX; ++m) {
                    const float x = vload_at(row(sb[v], m), moff[m] + ic4);
                    cs[v][m] = OUT ? x + away : x;
                }
        };
        // lane = reference: every lane's reference (lt, ls) against the candidates whose rows are in LDS,
        // c < c1, read back two at a time as broadcasts.  (From scalar loads the subtractions have an SGPR
        // operand and issue at half rate; the 15-neighbour lists of 410 chunks of 1 159 points took 1 302 us
        // that way against 1 044, the four-neighbour sets the same time.)
        auto scan_rows = [&](int c1, const float (&lt)[DT], const float (&ls)[V][DX]) {
            for (int c = 0; c < c1; c += 2) {
                float rr[2][RW], dtp[2];
                read_row(c, rr[0]);
                read_row(min(c + 1, kWave - 1), rr[1]);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    dtp[u] = absdiff(rr[u][0], lt[0]);
#pragma unroll
                    for (int m = 1; m < DT; ++m)
                        dtp[u] = fmaxf(dtp[u], absdiff(rr[u][m], lt[m]));
                }
                if (c + 1 >= c1)
                    dtp[1] = kInf;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    float dj[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        float d = absdiff(rr[u][DT + v * DX], ls[v][0]);
#pragma unroll
                        for (int m = 1; m < DX; ++m)
                            d = fmaxf(d, absdiff(rr[u][DT + v * DX + m], ls[v][m]));
                        dj[u] = fmaxf(dtp[u], d);
                    }
                    if (ballot(fminf(dj[0], dj[1]) < cur(v))) {
                        keep_branch();
                        insert(v, dj[0]);
                        insert(v, dj[1]);
                    }
                }
            }
        };
        // the same for block b, whose candidates take the place of the references' rows meanwhile
        auto scan_block = [&](int b) {
            float ct[DT], cs[V][DX], own[RW], lt[DT], ls[V][DX];
            load_block(b, ct, cs);
            read_row(lane, own);
#pragma unroll
            for (int m = 0; m < DT; ++m)
                lt[m] = own[m];
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int m = 0; m < DX; ++m)
                    ls[v][m] = own[DT + v * DX + m];
            store_row(ct, cs);
            scan_rows(min(kWave, n - b * kWave), lt, ls);
            store_row(lt, ls);
        };

        // the block's own points first (with a ragged last block, the block before it too, so
        // that every reference starts with a radius)
        const int ob0 = (blk > 0 && n - blk * kWave < kWave) ? blk - 1 : blk;
        const int e0 = min(n, (blk + 1) * kWave);
        const int nref = max(0, min(RPW, n - r0));
        if constexpr (W > 0) {
            // each group of RPW lanes takes every W-th candidate; the groups' lists are merged
            constexpr int U = 4;                           // candidates in flight per lane
            for (int j0 = ob0 * kWave; j0 < e0; j0 += U * W) {
                float dj[U][V];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int j = j0 + u * W + lane / RPW;
                    const uint32_t j4 = (uint32_t)min(j, e0 - 1) * 4u;
                    float dtp = absdiff(rt[0], vload_at(row(tb, 0), moff[0] + j4));
#pragma unroll
                    for (int m = 1; m < DT; ++m)
                        dtp = fmaxf(dtp, absdiff(rt[m], vload_at(row(tb, m), moff[m] + j4)));
                    dtp = j < e0 ? dtp : kInf;
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        float d = absdiff(rs[v][0], vload_at(row(sb[v], 0), moff[0] + j4));
#pragma unroll
                        for (int m = 1; m < DX; ++m)
                            d = fmaxf(d, absdiff(rs[v][m], vload_at(row(sb[v], m), moff[m] + j4)));
                        dj[u][v] = fmaxf(dtp, d);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        insert(v, dj[u][v]);
            }
#pragma unroll
            for (int o = RPW; o < kWave; o <<= 1)
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    float other[KP1];
#pragma unroll
                    for (int s = 0; s < KP1; ++s)
                        other[s] = __shfl_xor(best[v][s], o, 64);
#pragma unroll
                    for (int s = 0; s < KP1; ++s)
                        if (s >= fill)
                            insert_sorted<KP1>(best[v], other[s]);
                }
            store_row(rt, rs);
        } else {
            store_row(rt, rs);
            scan_rows(nref, rt, rs);
            if (ob0 < blk)
                scan_block(ob0);
            else
                store_radii();
        }
        unsigned long long ev = (unsigned long long)(e0 - ob0 * kWave) * (unsigned long long)nref;

        // distance of the lane's reference from a box (-inf: inside, or not a number)
        auto box_dist = [&](const float (&lo)[DY], const float (&hi)[DY]) {
            float g = -kInf;
#pragma unroll
            for (int m = 0; m < DY; ++m)
                g = fmaxf(g, fmaxf(lo[m] - rt[1 + m], rt[1 + m] - hi[m]));
            return g;
        };
        // boxes of the 64 blocks from b0, one per lane, and their distances from the references' own box
        float blo[DY], bhi[DY];
        if (nb > 1)
#pragma unroll
            for (int m = 0; m < DY; ++m) {
                blo[m] = uload(bx + (int64_t)(2 * m) * nb + blk);
                bhi[m] = uload(bx + (int64_t)(2 * m + 1) * nb + blk);
                if (W > 0) {
                    // the box of the wave's own references, which every group of RPW lanes holds
                    float lo = rt[1 + m], hi = rt[1 + m];
#pragma unroll
                    for (int o = 1; o < RPW; o <<= 1) {
                        lo = fminf(lo, __shfl_xor(lo, o, 64));
                        hi = fmaxf(hi, __shfl_xor(hi, o, 64));
                    }
                    if (blo[m] > -kInf && bhi[m] < kInf) {   // else: unbounded, or not numbers
                        blo[m] = readlane_f(lo, 0);
                        bhi[m] = readlane_f(hi, 0);
                    }
                }
            }
        auto load_boxes = [&](int b0, float (&lo)[DY], float (&hi)[DY]) {
            const uint32_t o = (uint32_t)min(b0 + lane, nb - 1) * 4u;
            float g = -kInf;
#pragma unroll
            for (int m = 0; m < DY; ++m) {
                lo[m] = vload_at(bx + (int64_t)(2 * m) * nb, o);
                hi[m] = vload_at(bx + (int64_t)(2 * m + 1) * nb, o);
                g = fmaxf(g, fmaxf(lo[m] - bhi[m], blo[m] - hi[m]));
            }
            return g;
        };
        // with W waves to a block the first 64 blocks' boxes stay in registers
        float lo0[DY], hi0[DY], g0 = 0.0f;
        if (W > 0 && nb > 1)
            g0 = load_boxes(0, lo0, hi0);
        auto boxes = [&](int b0, float (&lo)[DY], float (&hi)[DY]) {
            if (W == 0 || b0 > 0)
                return load_boxes(b0, lo, hi);
#pragma unroll
            for (int m = 0; m < DY; ++m) {
                lo[m] = lo0[m];
                hi[m] = hi0[m];
            }
            return g0;
        };
        auto box_of = [&](int c, const float (&lo)[DY], const float (&hi)[DY], float (&tlo)[DY], float (&thi)[DY]) {
#pragma unroll
            for (int m = 0; m < DY; ++m) {
                tlo[m] = readlane_f(lo[m], c);
                thi[m] = readlane_f(hi[m], c);
            }
        };

        // the other blocks that some reference's current radius reaches
        auto visit_block = [&](int b, const float (&tlo)[DY], const float (&thi)[DY]) {
            uint64_t todo = ballot(valid && !(box_dist(tlo, thi) >= curmax()));
            const int t0 = b * kWave, t1 = min(n, t0 + kWave);
            const int reach = __builtin_popcountll(todo);
            if (reach >= kDense) {
                ev += (unsigned long long)nref * (unsigned long long)(t1 - t0);
                scan_block(b);
                return;
            }
            if (reach == 0)
                return;
            ev += (unsigned long long)reach * (unsigned long long)(t1 - t0);
            float ct[DT], cs[V][DX];
            load_block(b, ct, cs);
            // lane = candidate: a candidate below a reference's radius is moved to the reference's
            // lane, where it waits in `pend` until the block is done (or a second one arrives)
            float pend[V];
#pragma unroll
            for (int v = 0; v < V; ++v)
                pend[v] = kInf;
            bool dirty = false;
            do {
                const int r = __builtin_ctzll(todo);
                todo = clear_bit(todo, r);
                float rr[RW];
                read_row(r, rr);
                float dtp = absdiff(rr[0], ct[0]);
#pragma unroll
                for (int m = 1; m < DT; ++m)
                    dtp = fmaxf(dtp, absdiff(rr[m], ct[m]));
                float dj[V];
                uint64_t hm[V], any = 0;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    float d = absdiff(rr[DT + v * DX], cs[v][0]);
#pragma unroll
                    for (int m = 1; m < DX; ++m)
                        d = fmaxf(d, absdiff(rr[DT + v * DX + m], cs[v][m]));
                    dj[v] = fmaxf(dtp, d);
                    hm[v] = ballot(dj[v] < rr[DT + V * DX + v]);
                    any |= hm[v];
                }
                if (any == 0)
                    continue;
                keep_branch();
                dirty = true;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    uint64_t hit = hm[v];
                    bool first = true;
                    while (hit != 0) {
                        keep_branch();
                        if (!first) {
                            insert(v, pend[v]);
                            pend[v] = kInf;
                            const float ut = readlane_f(cur(v), r);
                            hit &= ballot(dj[v] < ut);
                            if (hit == 0)
                                break;
                        }
                        const int c = __builtin_ctzll(hit);
                        hit &= hit - 1;
                        pend[v] = writelane_f(pend[v], readlane_f(dj[v], c), r);
                        first = false;
                    }
                }
            } while (todo != 0);
            if (dirty) {
#pragma unroll
                for (int v = 0; v < V; ++v)
                    insert(v, pend[v]);
                store_radii();
            }
        };
        if (nb > 1) {
            // Blocks are visited in four sweeps by their box's distance from the references' box,
            // nearer ones first, so that radii shrink before the farther blocks are tested.  The
            // limits are shares of the largest radius at the sweep's start; a block enters in the
            // sweep whose range its distance falls in, if the radii still reach it then.
            float lim = -kInf;
            for (int sw = 0; sw < 4; ++sw) {
                float cm = wave_max(curmax());
                const float share = sw == 0 ? 0.05f : (sw == 1 ? 0.15f : 0.4f);
                const float nlim = sw == 3 ? kInf : fmaxf(lim, share * cm);
                if (nlim == lim)
                    continue;
                for (int b0 = 0; b0 < nb; b0 += kWave) {
                    float lo[DY], hi[DY];
                    const float g = boxes(b0, lo, hi);
                    const int b = b0 + lane;
                    uint64_t want = ballot(b < nb && (b < ob0 || b > blk) && g >= lim && g < nlim && !(g >= cm));
                    if (want == 0)
                        continue;
                    do {
                        const int c = __builtin_ctzll(want);
                        want &= want - 1;
                        float tlo[DY], thi[DY];
                        box_of(c, lo, hi, tlo, thi);
                        visit_block(b0 + c, tlo, thi);
                    } while (want != 0);
                    cm = wave_max(curmax());
                }
                lim = nlim;
            }
        }
        float eps[V];
#pragma unroll
        for (int v = 0; v < V; ++v)
            eps[v] = cur(v);
        const float em = curmax();

        // ---- pass 2: lane = candidate, references uniform from this wave's LDS rows (which hold the
        // final radii); the three strict comparisons are wave ballots, counted on the SALU.  Bound by
        // issue: with four chunks at (3, 3) a step of 64 candidates is 45 VALU (28 of them at half rate), 28 SALU
        // and five LDS reads, 171 clocks per SIMD; the two-to-a-register counts took 11 SALU off it
        // (30 windows x 101 chunks of 1 000 to 50 000 points: 119.0 -> 110.6 ms; 94.1 with three chunks
        // and six waves).
        constexpr int NC = V + (V + 1) / 2;
        uint32_t accP[V], accTP[V], accPS[V];
        uint32_t packed[NC];                              // counts since the last unpack(), 16 bits each
        int counted = 0;                                  // candidates counted since then, at most 65 535
#pragma unroll
        for (int v = 0; v < V; ++v)
            accP[v] = accTP[v] = accPS[v] = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            packed[c] = 0;
        auto unpack = [&]() {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                accP[v] += packed[v] & 0xffffu;
                accTP[v] += packed[v] >> 16;
                accPS[v] += v % 2 == 0 ? packed[V + v / 2] & 0xffffu : packed[V + v / 2] >> 16;
            }
#pragma unroll
            for (int c = 0; c < NC; ++c)
                packed[c] = 0;
            counted = 0;
        };
        unsigned long long evaluated2 = 0;                // candidate-reference pairs examined in pass 2
        // Pre-embedded points may be infinite or no numbers: a coordinate without a difference says nothing
        // about its pair (fmaxf passes it over), but a pair without any in one space is outside the balls of
        // both, so there n_TP and n_PS are taken from both spaces' comparisons.  (The larger of the distances
        // as a maximum that keeps a NaN, v_maximum3_f32, was 1 to 2 % slower.)
        // counts of the references in todo over NS blocks of candidates
        auto count = [&](uint64_t todo, auto ns, const float (*ct)[DT], const float (*cs)[V][DX]) {
            constexpr int NS = decltype(ns)::value;
            // the counts of every reference in its lane, two to a register: n_P | n_TP << 16 of each
            // variant, then the variants' n_PS in pairs
            uint32_t t[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c)
                t[c] = 0;
            while (todo != 0) {
                const int r = __builtin_ctzll(todo);
                todo = clear_bit(todo, r);
                float rr[RW];
                read_row(r, rr);
                uint32_t sP[V], sTP[V], sPS[V];
#pragma unroll
                for (int v = 0; v < V; ++v)
                    sP[v] = sTP[v] = sPS[v] = 0;
#pragma unroll
                for (int sl = 0; sl < NS; ++sl) {
                    float dp = absdiff(rr[1], ct[sl][1]);
#pragma unroll
                    for (int m = 2; m < DT; ++m)
                        dp = fmaxf(dp, absdiff(rr[m], ct[sl][m]));
                    const float dt = absdiff(rr[0], ct[sl][0]);
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        float ds = absdiff(rr[DT + v * DX], cs[sl][v][0]);
#pragma unroll
                        for (int m = 1; m < DX; ++m)
                            ds = fmaxf(ds, absdiff(rr[DT + v * DX + m], cs[sl][v][m]));
                        const float er = rr[DT + V * DX + v];
                        const uint64_t in_p = ballot(dp < er);
                        sP[v] += (uint32_t)__builtin_popcountll(in_p);
                        sTP[v] += (uint32_t)__builtin_popcountll(OUT ? in_p & ballot(dt < er) : ballot(fmaxf(dt, dp) < er));
                        sPS[v] += (uint32_t)__builtin_popcountll(OUT ? in_p & ballot(ds < er)
                                                                      : ballot(fmaxf(dp, ds) < er));
                    }
                }
#pragma unroll
                for (int v = 0; v < V; ++v)
                    t[v] = writelane(t[v], pack16(sP[v], sTP[v]), r);
#pragma unroll
                for (int v = 0; v < V; v += 2)
                    t[V + v / 2] = writelane(t[V + v / 2], v + 1 < V ? pack16(sPS[v], sPS[v + 1]) : sPS[v], r);
            }
#pragma unroll
            for (int c = 0; c < NC; ++c)
                packed[c] += t[c];
            counted += kWave * NS;
            if (counted > 65535 - kWave * SLOTS)
                unpack();
        };
        auto evaluate = [&](uint64_t todo, int b) {
            evaluated2 += (unsigned long long)__builtin_popcountll(todo) * (unsigned long long)min(kWave, n - b * kWave);
        };
        if (nb > 1) {
            const float emw = wave_max(em);
            for (int b0 = 0; b0 < nb; b0 += kWave) {
                float lo[DY], hi[DY];
                const float g = boxes(b0, lo, hi);
                uint64_t want = ballot(b0 + lane < nb && !(g >= emw));
                while (want != 0) {
                    // the next SLOTS blocks that some reference reaches, counted together: a
                    // reference's row is read once for them
                    float ct[SLOTS][DT], cs[SLOTS][V][DX];
                    uint64_t todo = 0;
                    int used = 0, b = 0;
#pragma unroll
                    for (int sl = 0; sl < SLOTS; ++sl) {
                        uint64_t m = 0;
                        while (want != 0 && m == 0) {
                            const int c = __builtin_ctzll(want);
                            want &= want - 1;
                            float tlo[DY], thi[DY];
                            box_of(c, lo, hi, tlo, thi);
                            m = ballot(valid && !(box_dist(tlo, thi) >= em));
                            b = b0 + c;
                        }
                        if (m != 0)
                            used = sl + 1;
                        todo |= m;
                        load_block(b, ct[sl], cs[sl]);
                        // unused: outside every target-past ball; with one infinite coordinate only, an
                        // infinite reference would pass it over and take the block's points again
                        if (m == 0)
#pragma unroll
                            for (int x = 1; x < (OUT ? DT : 2); ++x)
                                ct[sl][x] = kInf;
                        evaluate(m, b);
                    }
                    if (used > 0)
                        count(todo, std::integral_constant<int, SLOTS>{}, ct, cs);
                }
            }
        } else if (nref > 0) {
            float ct[1][DT], cs[1][V][DX];
            load_block(0, ct[0], cs[0]);
            evaluate(ballot(valid), 0);
            count(ballot(valid), std::integral_constant<int, 1>{}, ct, cs);
        }

        unpack();

        // ---- per-point digamma terms of eq. 9, summed over the block in fixed order; self is at
        // distance 0 in every space and was counted iff its radius is positive
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const uint32_t self = eps[v] > 0.0f ? 1u : 0u;
            const int nP = (int)(accP[v] - self), nTP = (int)(accTP[v] - self), nPS = (int)(accPS[v] - self);
            double term = 0.0;
            if (valid)
                term = psi_of_count(nP) - psi_of_count(nTP) - psi_of_count(nPS);
            const double sum = wave_sum<RPW>(term);
            if (W > 0) {
                if (lane == 0)
                    wsum[v][threadIdx.x / kWave] = sum;
            } else if (lane == 0 && v < cnt) {
                a.partial[pb[v] + blk] = sum;
            }
            if constexpr (OUT) {
                const int64_t out = uload_l(reinterpret_cast<const int64_t *>(w0 + offsetof(ChunkDesc, out)));
                const int64_t perm = uload_l(reinterpret_cast<const int64_t *>(w0 + offsetof(ChunkDesc, perm)));
                if (out >= 0 && valid) {
                    // per-point outputs go to the point's index before ordering
                    int o = perm >= 0 ? order_at(a.perm_base + perm, n, i) : i;
                    if (o < 0 || o >= n)         // keep writes inside the chunk's output range regardless
                        o = i;
                    if (a.lte_out != nullptr)
                        a.lte_out[out + o] = psi_of_count(k - 1) + term;
                    if (a.eps_out != nullptr) {
                        a.eps_out[out + o] = eps[v];
                        a.cnt_out[out + o] = nP;
                        a.cnt_out[a.cnt_stride + out + o] = nTP;
                        a.cnt_out[2 * a.cnt_stride + out + o] = nPS;
                    }
                }
            }
        }
        if (W > 0) {
            // the waves' sums in the order of the butterfly that a whole wave's lanes go through
            __syncthreads();
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (threadIdx.x == 0 && v < cnt) {
                    double s[W > 0 ? W : 1];
#pragma unroll
                    for (int x = 0; x < W; ++x)
                        s[x] = wsum[v][x];
#pragma unroll
                    for (int o = 1; o < W; o <<= 1)
#pragma unroll
                        for (int x = 0; x < W; x += 2 * o)
                            s[x] += s[x + o];
                    a.partial[pb[v] + blk] = s[0];
                }
        }
        work1 += ev * (unsigned long long)cnt;
        work2 += evaluated2 * (unsigned long long)cnt;
        shared1 += ev;
        shared2 += evaluated2;
        if (W > 0)
            break;
    }
    // measurement: one pair of counter updates per wave, after its last item
    if (a.work != nullptr && lane == 0) {
        atomicAdd(a.work, work1);
        atomicAdd(a.work + 1, work2);
        atomicAdd(a.work + 2, shared1);
        atomicAdd(a.work + 3, shared2);
    }
}

// W waves to a block (W = 0: persistent waves, a block each).
template <int DY, int DX, int KP1, bool GENERIC, int SLOTS, int W>
__global__ void __launch_bounds__((W > 0 ? W : kMaxWavesPerWG) * 64) search_kernel(SearchArgs a)
{
    block_search<DY, DX, 1, KP1, GENERIC, SLOTS, true, W>(a);
}

// Waves per SIMD that a set's kernel is held to: the passes wait for LDS rows and issue slots of other
// pipes, and another wave fills them.  Six waves (85 VGPRs) where they cost a few spills at most: at
// (3, 3), three chunks, against five 100.4 to 94.1 ms on 30 windows x 101 chunks of 1 000 to 50 000
// points, seven 108 ms; at (3, 2) 8.49 to 8.08 ms on 8 windows x 61 chunks of 20 000 points.  With 14
// coordinates and more six cost more spills than they hide: (4, 3) 15.5 ms at five, 16.9 ms at six.
constexpr int sets_waves(int d_y, int d_x, int v, int w)
{
    return w > 0 ? 1 : (1 + d_y + v * d_x >= 14 ? 5 : 6);
}

template <int DY, int DX, int V, int SLOTS, int W>
__global__ void __launch_bounds__((W > 0 ? W : kMaxWavesPerWG) * 64)
    __attribute__((amdgpu_waves_per_eu(sets_waves(DY, DX, V, W), 8))) search_sets_kernel(SearchArgs a)
{
    block_search<DY, DX, V, 5, false, SLOTS, false, W>(a);
}

typedef void (*search_fn)(SearchArgs);

// The kernel of each pair of embedding dimensions; KERNEL(A, B) names it.
#define TE_SEARCH_KERNELS(KERNEL)                                               \
    static const search_fn fns[kMaxDimY][kMaxDimX] = {                          \
        {KERNEL(1, 1), KERNEL(1, 2), KERNEL(1, 3), KERNEL(1, 4)},               \
        {KERNEL(2, 1), KERNEL(2, 2), KERNEL(2, 3), KERNEL(2, 4)},               \
        {KERNEL(3, 1), KERNEL(3, 2), KERNEL(3, 3), KERNEL(3, 4)},               \
        {KERNEL(4, 1), KERNEL(4, 2), KERNEL(4, 3), KERNEL(4, 4)},               \
    };                                                                          \
    if (d_y < 1 || d_y > kMaxDimY || d_x < 1 || d_x > kMaxDimX)                 \
        return nullptr;                                                         \
    return fns[d_y - 1][d_x - 1]

// Single chunks with lists of CAP - 1 neighbours at most (ANYK) or exactly.
template <int CAP, bool ANYK, int SLOTS, int W>
search_fn pick_single(int d_y, int d_x)
{
#define TE_KERNEL(A, B) search_kernel<A, B, CAP, ANYK, SLOTS, W>
    TE_SEARCH_KERNELS(TE_KERNEL);
#undef TE_KERNEL
}

}  // namespace

// One source file each (they compile side by side); nullptr where there is no kernel.
search_fn pick_search_sets(int d_y, int d_x, int slots, int w);              // te_search_sets.hip: k = 4
search_fn pick_search_small_k(int d_y, int d_x, int k, int w);               // te_search_small_k.hip: k <= 8
search_fn pick_search_large_k(int d_y, int d_x, int w);                      // te_search_large_k.hip: k <= kMaxK

}  // namespace te

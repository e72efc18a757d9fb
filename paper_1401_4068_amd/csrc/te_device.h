// te_device.h -- device helpers shared by the kernel sources of libte (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "te_internal.h"

namespace te {
namespace {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) float cfloat_t;
typedef const __attribute__((address_space(4))) int32_t cint_t;
typedef const __attribute__((address_space(4))) int64_t cint64_t;
typedef const __attribute__((address_space(4))) f4v __attribute__((aligned(4))) cf4_t;

// Wave-uniform loads through the constant address space: the address is the
// same in every lane, so these become scalar (SMEM) loads into SGPRs.  Only
// scalar and vector-typed values are loaded this way (aggregate copies would
// be lowered to vector-memory loads).
__device__ __forceinline__ float uload(const float *p) { return *(cfloat_t *)p; }
// four at a 32-bit byte offset from a wave-uniform base: one SGPR offset shared by
// several bases, so the loads need no 64-bit address arithmetic
__device__ __forceinline__ f4v uload4_at(const float *p, uint32_t byte_off)
{
    typedef const __attribute__((address_space(4))) char cchar_t;
    return *(cf4_t *)((cchar_t *)p + byte_off);
}
// per-lane load at a 32-bit byte offset from a wave-uniform base: the base stays in
// SGPRs and the offset in one VGPR (no 64-bit address per lane)
__device__ __forceinline__ float vload_at(const float *p, uint32_t byte_off)
{
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(p) + byte_off);
}
__device__ __forceinline__ int32_t uload_i(const int32_t *p) { return *(cint_t *)p; }
__device__ __forceinline__ int64_t uload_l(const int64_t *p) { return *(cint64_t *)p; }

// Compiler barrier that keeps a uniform branch a branch (a block containing it
// cannot be speculated and if-converted into selects).
__device__ __forceinline__ void keep_branch() { asm volatile("" ::: "memory"); }

constexpr float kInf = __builtin_inff();

__device__ __forceinline__ float absdiff(float a, float b) { return __builtin_fabsf(a - b); }

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// psi(n + 1) = -gamma + H_n for integer n >= 0 in float64: upward recurrence
// psi(x) = psi(x + 1) - 1/x to x >= 16, then the asymptotic (Stirling-type)
// series psi(x) ~ ln x - 1/(2x) - sum_j B_2j / (2j x^2j) through B_10
// (Abramowitz & Stegun 6.3.18); truncation error < 1e-16 at x >= 16.
// Not inlined: its float64 constants (and those of log) would otherwise be
// hoisted out of the persistent work loop and held in VGPRs for the whole
// search, costing waves per SIMD.
__device__ __attribute__((noinline)) double psi_of_count(int n)
{
    double x = (double)n + 1.0;
    double shift = 0.0;
    while (x < 16.0) {
        shift -= 1.0 / x;
        x += 1.0;
    }
    const double r = 1.0 / x;
    const double r2 = r * r;
    const double series =
        r2 * (1.0 / 12 - r2 * (1.0 / 120 - r2 * (1.0 / 252 - r2 * (1.0 / 240 - r2 * (1.0 / 132)))));
    return log(x) - 0.5 * r - series + shift;
}

// Fixed-order butterfly sum over the 64 lanes (same order on every call), neighbouring lanes
// first: LANES < 64 gives every aligned group of LANES lanes the sum that is its part of the whole.
template <int LANES = kWave>
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 1; o < LANES; o <<= 1)
        v += __shfl_xor(v, o, 64);
    return v;
}

// Per-chunk coordinate base pointers (wave-uniform).
template <int DY, int DX>
struct Coords {
    static constexpr int D = 1 + DY + DX;
    const float *p[D];
    __device__ __forceinline__ Coords(const float *base, const ChunkDesc &c)
    {
#pragma unroll
        for (int m = 0; m < D; ++m)
            p[m] = (m < 1 + DY) ? base + c.tp + (int64_t)m * c.geo : base + c.s + (int64_t)(m - 1 - DY) * c.geo;
    }
};

// Joint, target-future, target-past and source-past distances of one pair.
template <int DY, int DX>
struct PairDist {
    float t, p, s;
};

template <int DY, int DX>
__device__ __forceinline__ PairDist<DY, DX> pair_dist(const float (&a)[1 + DY + DX], const float (&b)[1 + DY + DX])
{
    PairDist<DY, DX> d;
    d.t = absdiff(a[0], b[0]);
    float p = absdiff(a[1], b[1]);
#pragma unroll
    for (int m = 2; m < 1 + DY; ++m)
        p = fmaxf(p, absdiff(a[m], b[m]));
    float s = absdiff(a[1 + DY], b[1 + DY]);
#pragma unroll
    for (int m = 2 + DY; m < 1 + DY + DX; ++m)
        s = fmaxf(s, absdiff(a[m], b[m]));
    d.p = p;
    d.s = s;
    return d;
}

template <int DY, int DX, int RW>
__device__ __forceinline__ PairDist<DY, DX> pair_dist_row(const float (&a)[RW], const float (&b)[1 + DY + DX])
{
    float t[1 + DY + DX];
#pragma unroll
    for (int m = 0; m < 1 + DY + DX; ++m)
        t[m] = a[m];
    return pair_dist<DY, DX>(t, b);
}

// v_writelane_b32: returns old with lane `lane` replaced by the uniform value v.
__device__ __forceinline__ uint32_t writelane(uint32_t old, uint32_t v, int lane)
{
    // gfx9 allows one SGPR source per VALU op, so the lane select goes in M0.
    asm("v_writelane_b32 %0, %1, m0" : "+v"(old) : "s"(v), "{m0}"(lane));
    return old;
}

// One scalar instruction each: the SALU issues one in four clocks per SIMD and is what the
// counting loop waits for.  m without its bit r; and lo | hi << 16 of values below 2^16.
__device__ __forceinline__ uint64_t clear_bit(uint64_t m, int r)
{
    asm("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(r));
    return m;
}
__device__ __forceinline__ uint32_t pack16(uint32_t lo, uint32_t hi)
{
    uint32_t d;
    asm("s_pack_ll_b32_b16 %0, %1, %2" : "=s"(d) : "s"(lo), "s"(hi));
    return d;
}
__device__ __forceinline__ float readlane_f(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ float writelane_f(float old, float v, int lane)
{
    return __builtin_bit_cast(float, writelane(__builtin_bit_cast(uint32_t, old), __builtin_bit_cast(uint32_t, v), lane));
}

// Entry i of the order map of a space of n points: 16 bits wide up to kSortLds points (the
// other half of the map's n words then holds the block boxes), 32 bits above.
__device__ __forceinline__ int order_at(const int32_t *map, int n, int i)
{
    return n <= kSortLds ? (int)reinterpret_cast<const uint16_t *>(map)[i] : map[i];
}

// Middle one of three (one v_med3_u32).
__device__ __forceinline__ uint32_t med3_u32(uint32_t a, uint32_t b, uint32_t c)
{
    return max(min(a, b), min(max(a, b), c));
}

// Sorted-list insertion of x into the KP1 smallest values b[0] <= ... <= b[KP1-1]:
// from the top down, bi' = med3(b(i-1), bi, x), then b0' = min(b0, x).  Each
// step reads only entries not yet updated, so the list is rewritten in place
// (KP1 VALU ops, no copies).  Leaves the list unchanged when x >= b[KP1-1], so
// it can run on every lane of the wave.  All values are non-negative floats
// (+0 .. +inf) or no numbers, taken by their bit patterns, which order like
// unsigned integers: one that is no number is beyond every other (the float
// median would take it for the smallest).
template <int KP1>
__device__ __forceinline__ void insert_sorted(float (&b)[KP1], float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
#pragma unroll
    for (int i = KP1 - 1; i >= 1; --i)
        b[i] = __builtin_bit_cast(float, med3_u32(__builtin_bit_cast(uint32_t, b[i - 1]),
                                                  __builtin_bit_cast(uint32_t, b[i]), u));
    b[0] = __builtin_bit_cast(float, min(__builtin_bit_cast(uint32_t, b[0]), u));
}

template <int KP1, bool GENERIC>
__device__ __forceinline__ float kth(const float (&b)[KP1], int k)
{
    if (!GENERIC)
        return b[KP1 - 1];
    float r = b[0];
#pragma unroll
    for (int i = 1; i < KP1; ++i)
        r = (k == i) ? b[i] : r;
    return r;
}

// Work item -> chunk: the largest c with item_start[c] <= q (binary search on
// scalar loads).
__device__ __forceinline__ int find_chunk(const int32_t *item_start, int n_chunks, int q)
{
    int lo = 0, hi = n_chunks - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (uload_i(item_start + mid) <= q)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Largest of the wave's values, uniform: DPP row shifts, then the row broadcasts (no LDS).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x)
{
#define TE_STEP(ctrl, rows) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, 0xf, false))
    TE_STEP(0x111, 0xf);   // row_shr:1, 2, 4, 8: the row's largest in its last lane
    TE_STEP(0x112, 0xf);
    TE_STEP(0x114, 0xf);
    TE_STEP(0x118, 0xf);
    TE_STEP(0x142, 0xa);   // row_bcast:15
    TE_STEP(0x143, 0xc);   // row_bcast:31
#undef TE_STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)x, kWave - 1);
}
// The same for non-negative floats, whose bit patterns order like unsigned integers.
__device__ __forceinline__ float wave_max(float f)
{
    return __builtin_bit_cast(float, wave_max_u32(__builtin_bit_cast(uint32_t, f)));
}
// Inclusive sum over the lanes up to this one.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x)
{
#define TE_STEP(ctrl, rows) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, 0xf, false)
    TE_STEP(0x111, 0xf);   // row_shr:1, 2, 4, 8
    TE_STEP(0x112, 0xf);
    TE_STEP(0x114, 0xf);
    TE_STEP(0x118, 0xf);
    TE_STEP(0x142, 0xa);   // row_bcast:15
    TE_STEP(0x143, 0xc);   // row_bcast:31
#undef TE_STEP
    return x;
}

// Order-preserving unsigned image of a float (negative values reversed), and back.
__device__ __forceinline__ uint32_t orderable(float f)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_orderable(uint32_t u)
{
    return __builtin_bit_cast(float, (u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

// Box of a wave's 64 values: their smallest and largest, uniform; unbounded if one is no
// number (its distances then say nothing, so nothing may be skipped for them).
__device__ __forceinline__ void wave_box(float v, float *lo, float *hi)
{
    *lo = from_orderable(~wave_max_u32(~orderable(v != v ? -kInf : v)));
    *hi = from_orderable(wave_max_u32(orderable(v != v ? kInf : v)));
}

}  // namespace
}  // namespace te

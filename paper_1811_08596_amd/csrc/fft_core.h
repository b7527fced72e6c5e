// Device-side building blocks of the LDS-resident Stockham FFT passes (shared by the per-pass kernels in
// fft.hip, the fused, cache-resident kernels in fused.hip and the chunk-resident codec in chunk.hip).  Internal: nothing here is part of the C ABI.
#pragma once
#include "internal.h"
#include "stretches.h"

namespace fftsp {
namespace {

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// Several kernels compute the same transform: with small tiles and large ones, for uniform chunks and for tensors, the codec's
// own and the stage-level ones.  They have to agree bit for bit, so nothing is left to the compiler's choice of what becomes a
// fused multiply-add (the sources are compiled with -ffp-contract=off): every fused operation is written out.
// Of two products that meet, the second is rounded before the sum.  In a * b that is the one with the imaginary part of b: most
// twiddles, and all entries of the fine table, lie nearer the real axis, so it is the smaller one.
__device__ __forceinline__ float prod_sum(float a, float b, float c, float d) { return __fmaf_rn(a, b, c * d); }
__device__ __forceinline__ float prod_diff(float a, float b, float c, float d) { return __fmaf_rn(a, b, -(c * d)); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b)
{
    return make_float2(prod_diff(a.x, b.x, a.y, b.y), prod_sum(a.y, b.x, a.x, b.y));
}
// a * conj(b)
__device__ __forceinline__ float2 cmulc(float2 a, float2 b)
{
    return make_float2(prod_sum(a.x, b.x, a.y, b.y), prod_diff(a.y, b.x, a.x, b.y));
}

// exp(-2 pi i E / 2^22), E < 2^22
__device__ __forceinline__ float2 twiddle(const Tables& t, uint32_t E)
{
    return cmul(t.hi[E >> 11], t.lo[E & 2047u]);
}

template <int LOGT>
__device__ __forceinline__ int sw_idx(int i, int b)
{
    if constexpr (LOGT == 0)
        return i;
    else if constexpr (LOGT >= 4)
        return (i << LOGT) + (b ^ (i & 15));
    else
        return (i << LOGT) + (b ^ ((i >> (4 - LOGT)) & ((1 << LOGT) - 1)));
}

// multiply by -i (forward) or +i (inverse)
template <bool INV>
__device__ __forceinline__ float2 rot90(float2 a)
{
    return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

template <bool INV>
__device__ __forceinline__ void bf2(float2* v)
{
    float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

template <bool INV>
__device__ __forceinline__ void bf4(float2* v)
{
    float2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    float2 t2 = cadd(v[1], v[3]), t3 = rot90<INV>(csub(v[1], v[3]));
    v[0] = cadd(t0, t2);
    v[1] = cadd(t1, t3);
    v[2] = csub(t0, t2);
    v[3] = csub(t1, t3);
}

template <bool INV>
__device__ __forceinline__ void bf8(float2* v)
{
    const float c = 0.70710678118654752440f;
    float2 e[4] = {v[0], v[2], v[4], v[6]};
    float2 o[4] = {v[1], v[3], v[5], v[7]};
    bf4<INV>(e);
    bf4<INV>(o);
    // v[k], v[k+4] = e[k] +- W8^k o[k]; the odd powers of W8 are (1 -+ i) / sqrt(2) times a real factor
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    o[2] = rot90<INV>(o[2]);
    v[2] = cadd(e[2], o[2]);
    v[6] = csub(e[2], o[2]);
    const float2 o1 = INV ? make_float2(o[1].x - o[1].y, o[1].x + o[1].y) : make_float2(o[1].x + o[1].y, o[1].y - o[1].x);
    const float2 o3 = INV ? make_float2(-(o[3].x + o[3].y), o[3].x - o[3].y) : make_float2(o[3].y - o[3].x, -(o[3].x + o[3].y));
    v[1] = make_float2(__fmaf_rn(c, o1.x, e[1].x), __fmaf_rn(c, o1.y, e[1].y));
    v[5] = make_float2(__fmaf_rn(-c, o1.x, e[1].x), __fmaf_rn(-c, o1.y, e[1].y));
    v[3] = make_float2(__fmaf_rn(c, o3.x, e[3].x), __fmaf_rn(c, o3.y, e[3].y));
    v[7] = make_float2(__fmaf_rn(-c, o3.x, e[3].x), __fmaf_rn(-c, o3.y, e[3].y));
}

// 16 points: four radix-4 butterflies over n1 (elements n0, n0+4, n0+8, n0+12), the inner twiddles W16^(n0 k0),
// four radix-4 butterflies over n0; output k = k0 + 4 k1.  One LDS round trip where two radix-4 stages take two.
template <bool INV>
__device__ __forceinline__ void bf16(float2* v)
{
    const float c1 = 0.92387953251128674f, s1 = 0.38268343236508977f, h = 0.70710678118654752440f;
    float2 y[4][4];  // y[n0][k0]
#pragma unroll
    for (int n0 = 0; n0 < 4; ++n0) {
        float2 t[4] = {v[n0], v[n0 + 4], v[n0 + 8], v[n0 + 12]};
        bf4<INV>(t);
#pragma unroll
        for (int k0 = 0; k0 < 4; ++k0) y[n0][k0] = t[k0];
    }
    // W16^m = (cos(m pi/8), -sin(m pi/8)), conjugated for the inverse
    // y *= wr + i wi, forward; its conjugate, inverse; where the imaginary part is the larger one, as i y times wi - i wr
    auto rot = [&](int n0, int k0, float wr, float wi) __attribute__((always_inline)) {
        const float2 a = y[n0][k0];
        if (wr * wr >= wi * wi)
            y[n0][k0] = INV ? cmulc(a, make_float2(wr, wi)) : cmul(a, make_float2(wr, wi));
        else
            y[n0][k0] = INV ? cmulc(make_float2(a.y, -a.x), make_float2(wi, -wr)) : cmul(make_float2(-a.y, a.x), make_float2(wi, -wr));
    };
    rot(1, 1, c1, -s1);                // W^1
    rot(1, 2, h, -h);                  // W^2
    rot(1, 3, s1, -c1);                // W^3
    rot(2, 1, h, -h);                  // W^2
    y[2][2] = rot90<INV>(y[2][2]);     // W^4 = -i
    rot(2, 3, -h, -h);                 // W^6
    rot(3, 1, s1, -c1);                // W^3
    rot(3, 2, -h, -h);                 // W^6
    rot(3, 3, -c1, s1);                // W^9
#pragma unroll
    for (int k0 = 0; k0 < 4; ++k0) {
        float2 t[4] = {y[0][k0], y[1][k0], y[2][k0], y[3][k0]};
        bf4<INV>(t);
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) v[k0 + 4 * k1] = t[k1];
    }
}

template <int RL, bool INV>
__device__ __forceinline__ void butterfly(float2* v)
{
    if constexpr (RL == 1) bf2<INV>(v);
    if constexpr (RL == 2) bf4<INV>(v);
    if constexpr (RL == 3) bf8<INV>(v);
    if constexpr (RL == 4) bf16<INV>(v);
}

// log2 of the next stage's radix when `rem` binary stages remain: as few LDS round trips as a lane's sixteen
// points allow (radix 16 where the count is not a multiple of three).
__host__ __device__ constexpr int stage_radix_log(int rem)
{
    return rem <= 4 ? rem : (rem % 3 == 0 ? 3 : (rem == 5 ? 2 : 4));
}

// One Stockham stage of radix 2^RL on T = 2^LOGT interleaved R-point transforms.
// NS = product of the radices already applied.  tw[e] = exp(-2 pi i e / R).
// With fewer butterflies than lanes the last lanes have none.
template <int LOGR, int LOGT, int NT, bool INV, int NS_LOG, int RL>
__device__ __forceinline__ void fft_stage(float2* d, const float2* tw, int tid)
{
    constexpr int R = 1 << LOGR, T = 1 << LOGT, RHO = 1 << RL, NS = 1 << NS_LOG;
    constexpr int NBF = (R / RHO) * T;
    static_assert(NBF % NT == 0 || (NBF < NT && NBF % 64 == 0), "butterflies must divide evenly over the workgroup, or over some of its waves");
    constexpr int PER = NBF < NT ? 1 : NBF / NT;
    const bool on = NBF >= NT || tid < NBF;
    float2 v[PER][RHO];
    if (on) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int w = tid + q * NT, b = w & (T - 1), j = w >> LOGT;
#pragma unroll
            for (int t = 0; t < RHO; ++t) v[q][t] = d[sw_idx<LOGT>(j + t * (R / RHO), b)];
        }
    }
    __syncthreads();
    if (on) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int w = tid + q * NT, b = w & (T - 1), j = w >> LOGT;
            const int k = j & (NS - 1);
            if constexpr (NS > 1) {
#pragma unroll
                for (int t = 1; t < RHO; ++t) {
                    const float2 c = tw[(t * k) << (LOGR - NS_LOG - RL)];
                    v[q][t] = INV ? cmulc(v[q][t], c) : cmul(v[q][t], c);
                }
            }
            butterfly<RL, INV>(v[q]);
            const int base = ((j >> NS_LOG) << (NS_LOG + RL)) + k;
#pragma unroll
            for (int t = 0; t < RHO; ++t) d[sw_idx<LOGT>(base + t * NS, b)] = v[q][t];
        }
    }
    __syncthreads();
}

template <int LOGR, int LOGT, int NT, bool INV, int NS_LOG = 0>
__device__ __forceinline__ void run_fft(float2* d, const float2* tw, int tid)
{
    if constexpr (NS_LOG < LOGR) {
        constexpr int RL = stage_radix_log(LOGR - NS_LOG);
        fft_stage<LOGR, LOGT, NT, INV, NS_LOG, RL>(d, tw, tid);
        run_fft<LOGR, LOGT, NT, INV, NS_LOG + RL>(d, tw, tid);
    }
}

// The same, but the last stage leaves its outputs in registers: put(q, t, value) of row j + t * R / 2^RL, j = (tid + q * NT) / T, slot tid % T.
template <int LOGR, int LOGT, int NT, bool INV, int NS_LOG, typename Put>
__device__ __forceinline__ void run_fft_put(float2* d, const float2* tw, int tid, Put&& put)
{
    constexpr int RL = stage_radix_log(LOGR - NS_LOG);
    if constexpr (NS_LOG + RL < LOGR) {
        fft_stage<LOGR, LOGT, NT, INV, NS_LOG, RL>(d, tw, tid);
        run_fft_put<LOGR, LOGT, NT, INV, NS_LOG + RL>(d, tw, tid, static_cast<Put&&>(put));
    } else {
        constexpr int R = 1 << LOGR, T = 1 << LOGT, RHO = 1 << RL, PER = (R / RHO) * T / NT;
        static_assert(PER * NT == (R / RHO) * T, "butterflies for all lanes");
        float2 v[PER][RHO];
#pragma unroll
        for (int q = 0; q < PER; ++q)
#pragma unroll
            for (int t = 0; t < RHO; ++t) v[q][t] = d[sw_idx<LOGT>(((tid + q * NT) >> LOGT) + t * (R / RHO), tid & (T - 1))];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
#pragma unroll
            for (int t = 1; t < RHO; ++t) {
                const float2 c = tw[t * ((tid + q * NT) >> LOGT)];
                v[q][t] = INV ? cmulc(v[q][t], c) : cmul(v[q][t], c);
            }
            butterfly<RL, INV>(v[q]);
#pragma unroll
            for (int t = 0; t < RHO; ++t) put(q, t, v[q][t]);
        }
    }
}

// Sixteen transforms of N2 = 2^LOGN2 points, sixteen points a lane, in half of the LDS they would take as complex values: between
// the stages real and imaginary parts go through it one after the other.  The slots are eight pairs (rows k1 and their mirrors).
template <int LOGN2>
struct HalfTile {
    static constexpr int N2 = 1 << LOGN2, SLOTS = 16, PAIRS = 8, NT = N2, DK = N2 / 8;
    static constexpr size_t kLds = (size_t)N2 * (SLOTS * sizeof(uint32_t) + sizeof(float2));  // and the stage twiddles
    static constexpr int RL2 = stage_radix_log(LOGN2 - 3), RL3 = LOGN2 - 3 - RL2, LAST = RL3 ? RL3 : RL2;  // after a first stage of radix 8
    static_assert(RL3 == 0 || stage_radix_log(RL3) == RL3, "three stages at most");

    // Row i, place s of a component (places: the pairs' lower slots, then the upper ones) is word i * 16 + s with i >> 3 swizzled in, so that
    // 64 lanes have two words of every bank whether they hold neighbouring rows or rows eight apart.
    static __device__ __forceinline__ int swizzled(int word, int x) { return word ^ (x & 3) << 3; }
    static __device__ __forceinline__ int place(int slot) { return (slot & 1) * PAIRS + (slot >> 1); }
    // the first stage's output n of a butterfly of rows i + q * DK
    static __device__ __forceinline__ int first_output(int i, int t, int place) { return i * 128 + (t >> 1) * 32 + swizzled((t & 1) * 16 + place, i); }
    // Inputs n = q * RHO + t of a stage of radix RHO = 2^RL, and outputs of the second stage: slot tid % 16.
    static __device__ __forceinline__ int row_of(int tid, int q) { return (tid >> 4) + q * (N2 / 16); }
    template <int RL>
    static __device__ __forceinline__ int input(int tid, int n)
    {
        constexpr int RHO = 1 << RL;
        return at_row<N2 / RHO>(row_of(tid, n / RHO), n % RHO, place(tid & 15));
    }
    static __device__ __forceinline__ int second_output(int tid, int n)
    {
        const int i = row_of(tid, n >> RL2), t = n & ((1 << RL2) - 1);
        return swizzled((((i >> 3) << (3 + RL2)) + (i & 7)) * 16 + place(tid & 15), t) + t * 128;
    }
    // row i + t * STEP
    template <int STEP>
    static __device__ __forceinline__ int at_row(int i, int t, int place)
    {
        return swizzled(i * 16 + place, STEP >= 32 ? i >> 3 : (i >> 3) + t * (STEP / 8)) + t * STEP * 16;
    }
    template <typename To, typename From>
    static __device__ __forceinline__ void exchange(float* d, float2 (&v)[16], To&& to, From&& from)
    {
        float x[16];
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 16; ++n) d[to(n)] = v[n].x;
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 16; ++n) x[n] = d[from(n)];
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 16; ++n) d[to(n)] = v[n].y;
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 16; ++n) v[n] = make_float2(x[n], d[from(n)]);
    }
    // row(q): that of the q-th butterfly's first input
    template <bool INV, int NS_LOG, int RL, typename Row>
    static __device__ __forceinline__ void stage(float2 (&v)[16], const float2* tw, Row&& row)
    {
        constexpr int RHO = 1 << RL;
#pragma unroll
        for (int q = 0; q < 16 / RHO; ++q) {
            const int k = row(q) & ((1 << NS_LOG) - 1);
#pragma unroll
            for (int t = 1; t < RHO; ++t) {
                const float2 c = tw[(t * k) << (LOGN2 - NS_LOG - RL)];
                v[q * RHO + t] = INV ? cmulc(v[q * RHO + t], c) : cmul(v[q * RHO + t], c);
            }
            butterfly<RL, INV>(v + q * RHO);
        }
    }
};
// Which rows of a tile of mirrored rows a lane has: at(0) + q * N2/8 of one slot and at(1) + q * N2/8 of another, q and 7 - q of which are
// each other's mirrors: pair j's lower slot and its upper one, rows r and N2/8 - 1 - r.  Rows k1 = 0 and N1/2 (pair 0 of a chunk's first
// tile) are their own mirrors: of those a lane has both from the same slot, and the lane `alone` row 0's points 0 and N2/16, each with itself.
template <int LOGN2>
struct MirroredRows {
    static constexpr int DK = (1 << LOGN2) / 8;
    int at0, at1, upper0, upper1;
    bool alone;
    __device__ __forceinline__ MirroredRows(uint32_t pp, int r)
    {
        const bool self = pp == 0, lower = r >= DK / 2;
        alone = self && r == DK / 2;
        at0 = self && lower ? r - DK / 2 : r;
        at1 = self && lower ? (alone ? DK / 2 : DK + DK / 2 - r) : DK - 1 - r;
        upper0 = self && !lower ? 1 : 0;
        upper1 = self && lower ? 0 : 1;
    }
    __device__ __forceinline__ int at(int i) const { return i ? at1 : at0; }
    __device__ __forceinline__ int upper(int i) const { return i ? upper1 : upper0; }
};

// this workgroup's tile; at or above `total`: none
__device__ __forceinline__ uint32_t in_stretches(uint32_t total) { return stretch_tile(blockIdx.x, total); }
__device__ __forceinline__ uint32_t in_stretches(uint32_t total, uint32_t few) { return stretch_tile(blockIdx.x, total, few); }
__device__ __forceinline__ uint32_t in_turned_stretches(uint32_t total, uint32_t step) { return turned_tile(blockIdx.x, total, step); }

// Accesses that leave the caches to others (ONCE), for what the call does not touch again: whole calls choose, see kOnceBytes.
template <bool ONCE>
__device__ __forceinline__ void store_maybe_once(float4* p, float4 v)
{
    using F4 = float __attribute__((ext_vector_type(4)));
    if constexpr (ONCE)
        __builtin_nontemporal_store(F4{v.x, v.y, v.z, v.w}, reinterpret_cast<F4*>(p));
    else
        *p = v;
}
template <bool ONCE>
__device__ __forceinline__ float4 load_maybe_once(const float4* p)
{
    using F4 = float __attribute__((ext_vector_type(4)));
    if constexpr (ONCE) {
        const F4 v = __builtin_nontemporal_load(reinterpret_cast<const F4*>(p));
        return make_float4(v[0], v[1], v[2], v[3]);
    } else {
        return *p;
    }
}
template <bool ONCE>
__device__ __forceinline__ uint2 load_maybe_once(const uint2* p)
{
    using U2 = uint32_t __attribute__((ext_vector_type(2)));
    if constexpr (ONCE) {
        const U2 v = __builtin_nontemporal_load(reinterpret_cast<const U2*>(p));
        return make_uint2(v[0], v[1]);
    } else {
        return *p;
    }
}

// LDS stages run_fft takes for `rem` remaining levels
constexpr int lds_stages(int rem)
{
    int n = 0;
    while (rem > 0) {
        rem -= stage_radix_log(rem);
        ++n;
    }
    return n;
}

// the same, calling between(k) after LDS stage k (k = 0, 1, ...)
template <int LOGR, int LOGT, int NT, bool INV, int NS_LOG, int K = 0, typename Between>
__device__ __forceinline__ void run_fft_between(float2* d, const float2* tw, int tid, Between between)
{
    if constexpr (NS_LOG < LOGR) {
        constexpr int RL = stage_radix_log(LOGR - NS_LOG);
        fft_stage<LOGR, LOGT, NT, INV, NS_LOG, RL>(d, tw, tid);
        between(K);
        run_fft_between<LOGR, LOGT, NT, INV, NS_LOG + RL, K + 1>(d, tw, tid, between);
    }
}

template <int LOGR, int NT>
__device__ __forceinline__ void load_stage_twiddles(float2* tw, const Tables& tb, int tid)
{
    if constexpr (LOGR <= 11) {
        for (int e = tid; e < (1 << LOGR); e += NT) tw[e] = tb.hi[e << (11 - LOGR)];
    } else {
        for (int e = tid; e < (1 << LOGR); e += NT) tw[e] = twiddle(tb, (uint32_t)e << (22 - LOGR));
    }
}

// Neighbouring samples wherever they start: accesses of 8 and 16 bytes need an alignment of four.  Most tensors start at any multiple of
// four bytes, and lanes that move a float at a time touch every line many times.
using Floats2 = float __attribute__((ext_vector_type(2), aligned(4)));
using Floats4 = float __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float2 load_pair(const float* __restrict__ in, size_t gi, size_t n)
{
    if (gi + 1 < n) {
        const Floats2 v = *reinterpret_cast<const Floats2*>(in + gi);
        return make_float2(v[0], v[1]);
    }
    if (gi < n) return make_float2(in[gi], 0.f);
    return make_float2(0.f, 0.f);
}

// Where chunk c's samples live: elements [first, limit) of the gradient.
struct Span {
    size_t first, limit;
};
// Pairs at + t * step of a span of at most `all` of them, zeros behind its end.  No load stands in a branch but that of a pair cut in two,
// so that all are on their way together; those that do not exist read a table.
template <int N>
__device__ __forceinline__ void load_pairs(float2 (&v)[N], const float* __restrict__ in, const Span& sp, uint32_t all, uint32_t at, uint32_t step,
                                           const Tables& tb)
{
    const size_t left = sp.limit > sp.first ? sp.limit - sp.first : 0;
    const uint32_t whole = left >> 1 < all ? (uint32_t)(left >> 1) : all;
    const float* src = whole ? in + sp.first : reinterpret_cast<const float*>(tb.hi);
    Floats2 r[N];
    if (whole == all) {
#pragma unroll
        for (int t = 0; t < N; ++t) {
            r[t] = *reinterpret_cast<const Floats2*>(src + 2 * (size_t)(at + (uint32_t)t * step));
            v[t] = make_float2(r[t][0], r[t][1]);
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < N; ++t) {
        const uint32_t i = at + (uint32_t)t * step;
        r[t] = *reinterpret_cast<const Floats2*>(src + 2 * (size_t)(i < whole ? i : 0u));
    }
#pragma unroll
    for (int t = 0; t < N; ++t) v[t] = at + (uint32_t)t * step < whole ? make_float2(r[t][0], r[t][1]) : make_float2(0.f, 0.f);
    if (left & 1u) {
#pragma unroll
        for (int t = 0; t < N; ++t)
            if (at + (uint32_t)t * step == whole) v[t].x = in[sp.limit - 1];
    }
}

__device__ __forceinline__ void store_pair(float* __restrict__ out, size_t gi, size_t n, float2 v)
{
    if (gi + 1 < n)
        *reinterpret_cast<Floats2*>(out + gi) = Floats2{v.x, v.y};
    else if (gi < n)
        out[gi] = v.x;
}


// what a launch covers: samples [first, first + count), cut into chunks
__device__ __forceinline__ Span chunk_span(size_t first, size_t count, size_t c, size_t chunk_len)
{
    return Span{first + c * chunk_len, first + count};
}

// X[k] from a = Z[k], b = Z[M-k], w = W_L^k   (0 < k < M); times 2 half, a power of two
__device__ __forceinline__ float2 split_fwd(float2 a, float2 b, float2 w, float half = 0.5f)
{
    const float dr = half * (a.x - b.x), di = half * (a.y + b.y);
    return make_float2(__fmaf_rn(half, a.x + b.x, prod_sum(w.x, di, w.y, dr)),
                       __fmaf_rn(half, a.y - b.y, -prod_diff(w.x, dr, w.y, di)));
}

// 2 Z[k] from a = X[k], b = X[M-k], w = W_L^k  (the factor 1/2 is folded into the final 1/L)
__device__ __forceinline__ float2 split_inv(float2 a, float2 b, float2 w)
{
    const float er = a.x + b.x, ei = a.y - b.y;
    const float dr = a.x - b.x, di = a.y + b.y;
    const float orr = prod_sum(w.x, dr, w.y, di), oi = prod_diff(w.x, di, w.y, dr);  // conj(w) * d
    return make_float2(er - oi, ei + orr);
}


// --------------------------------------------------------------- two pass ---
// The two-pass kernels are persistent: a workgroup of 512 lanes walks a contiguous run of tiles and, while
// the LDS FFT of tile i runs, the global loads of tile i+1 are already in flight into registers.
//
// Twiddles outside the LDS stages are not gathered per element.  Along the index a lane walks, the exponent
// grows by a fixed step, so W^(e0 + j*step) = W^e0 * (W^step)^j: one table lookup for the base, one for the
// ratio, then a short recurrence that is re-anchored from the table every 8 steps; for the even/odd split the
// step is always 1/32 of a turn, so exact constants are used instead of a recurrence.

// Loop-invariant per-lane addresses (LDS swizzles, global offsets of 16 loads and 16 stores, four stages of
// butterfly indices) would otherwise be hoisted out of the persistent loop and held in ~100 VGPRs; making the
// lane id opaque once per iteration has them recomputed (a few integer ops) and keeps two workgroups per CU.
__device__ __forceinline__ int opaque_lane(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

constexpr int kNT = 512;   // lanes per workgroup in the two-pass kernels
constexpr int kLogE = 13;  // 8192 complex points (64 KiB) per tile
constexpr int kPer = (1 << kLogE) / kNT;
constexpr int kSplitStep = (16 * kNT) >> kLogE;  // 32nds of a turn between a lane's consecutive split twiddles
constexpr int kHistLdsWords = kHistBins / 2;  // 16-bit counters, two per word

// exp(-2 pi i q / 32), q = 0..15
__device__ constexpr float kW32re[16] = {1.0f, 0.98078528040323043f, 0.92387953251128674f, 0.83146961230254524f,
                                         0.70710678118654752f, 0.55557023301960223f, 0.38268343236508977f,
                                         0.19509032201612827f, 0.0f, -0.19509032201612827f, -0.38268343236508977f,
                                         -0.55557023301960223f, -0.70710678118654752f, -0.83146961230254524f,
                                         -0.92387953251128674f, -0.98078528040323043f};
__device__ constexpr float kW32im[16] = {-0.0f, -0.19509032201612827f, -0.38268343236508977f, -0.55557023301960223f,
                                         -0.70710678118654752f, -0.83146961230254524f, -0.92387953251128674f,
                                         -0.98078528040323043f, -1.0f, -0.98078528040323043f, -0.92387953251128674f,
                                         -0.83146961230254524f, -0.70710678118654752f, -0.55557023301960223f,
                                         -0.38268343236508977f, -0.19509032201612827f};

// The intermediate between the two passes is stored "paired": within each run of N1 values, row k1 and its
// mirror N1-k1 (the two rows the real-FFT split combines) sit next to each other,
//     position 2*k1   holds row k1        (k1 < N1/2)
//     position 2*k1+1 holds row N1-k1     (position 1 holds row N1/2, which like row 0 is its own mirror)
// so a pass-B tile of TB rows plus their mirrors is one contiguous run of 2*TB positions (128 bytes for TB = 8).
__device__ __forceinline__ uint32_t row_of_pos(uint32_t p, uint32_t N1)
{
    return (p & 1u) ? (p == 1u ? N1 / 2 : N1 - (p >> 1)) : (p >> 1);
}

// Two adjacent slots of one LDS row travel as one 16-byte value: the XOR swizzle keeps an even/odd slot pair
// adjacent (possibly swapped), so a pair is one 128-bit LDS access plus a conditional swap.
__device__ __forceinline__ float2 lo2(float4 v) { return make_float2(v.x, v.y); }
__device__ __forceinline__ float2 hi2(float4 v) { return make_float2(v.z, v.w); }
__device__ __forceinline__ float4 join(float2 a, float2 b) { return make_float4(a.x, a.y, b.x, b.y); }

template <int LOGT>
__device__ __forceinline__ void lds_store2(float2* d, int i, int b2, float4 v)
{
    static_assert(LOGT >= 1, "needs at least two slots per row");
    const int idx = sw_idx<LOGT>(i, b2);  // slot b2 (even); slot b2+1 lives at idx^1
    *reinterpret_cast<float4*>(d + (idx & ~1)) = (idx & 1) ? make_float4(v.z, v.w, v.x, v.y) : v;
}

template <int LOGT>
__device__ __forceinline__ float4 lds_load2(const float2* d, int i, int b2)
{
    static_assert(LOGT >= 1, "needs at least two slots per row");
    const int idx = sw_idx<LOGT>(i, b2);
    const float4 v = *reinterpret_cast<const float4*>(d + (idx & ~1));
    return (idx & 1) ? make_float4(v.z, v.w, v.x, v.y) : v;
}

// Which tile of its chunk work item `tile` is.  Workgroups walk runs of consecutive work items in step, so
// at any moment the chip would touch only every per_wg-th tile position of each chunk: a few fixed byte offsets
// of every row, i.e. a fraction of the memory channels.  Rotating the order by the chunk index spreads the
// offsets in flight over the whole row; the rotation is a multiple of 4, so aligned groups of up to 4 tiles stay together.
// (tiles is a power of two.)
__device__ __forceinline__ uint32_t tile_in_chunk(uint32_t tile, uint32_t tiles)
{
    return (tile + 4 * (tile / tiles)) & (tiles - 1);
}

// Tile run of a pass-A workgroup.  A pass-A tile is 64 bytes of every row it touches, half a 128-byte line;
// tiles 2m and 2m+1 share their lines.  Workgroups are dealt to the 8 XCDs round-robin by index, so workgroups
// b, b+8, ... share an L2: 2^glog of them walk the members of the same run of aligned tile groups in step, and
// each line crosses the fabric once.  The workgroup's tiles are t, t+2^glog, ... < tend.  Returns false if this
// workgroup has nothing to do.
__device__ __forceinline__ bool grouped_run(uint32_t b, uint32_t groups, uint32_t per_wg, int glog, uint32_t& t, uint32_t& tend)
{
    const uint32_t x = b & 7u, y = b >> 3, h = y & ((1u << glog) - 1u);
    const uint32_t rho = ((y >> glog) << 3) + x;  // which group of workgroups
    const uint32_t p0 = rho * per_wg;
    if (p0 >= groups) return false;
    const uint32_t p1 = p0 + per_wg < groups ? p0 + per_wg : groups;
    t = (p0 << glog) + h;
    tend = p1 << glog;
    return true;
}

// rows held by pair kp of a run of N1 paired positions: (kp, N1-kp), and (0, N1/2) for kp = 0
__device__ __forceinline__ uint32_t mirror_row(uint32_t kp, uint32_t N1) { return kp ? N1 - kp : N1 / 2; }

// The first radix-8 stage of an R-point Stockham chain, done in registers: a lane that holds rows j + t*R/8
// (t = 0..7) of two adjacent columns has all inputs of two butterflies, so the stage needs no LDS round trip and
// no barrier of its own.  The outputs go to rows 8j + t, where the next stage (NS = 8) reads them.
template <int LOGT, bool INV>
__device__ __forceinline__ void first_stage_store(float2* d, int j, int col_even, const float4 (&x)[8])
{
    float2 a[8], b[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        a[t] = lo2(x[t]);
        b[t] = hi2(x[t]);
    }
    bf8<INV>(a);
    bf8<INV>(b);
#pragma unroll
    for (int t = 0; t < 8; ++t) lds_store2<LOGT>(d, 8 * j + t, col_even, join(a[t], b[t]));
}

// rank key of a bin: the bit pattern of fl(re*re + fl(im*im)), sign bit masked (see key_of in codec.hip)
__device__ __forceinline__ uint32_t fft_key_of(float2 z)
{
    return __float_as_uint(__fmaf_rn(z.x, z.x, __fmul_rn(z.y, z.y))) & 0x7FFFFFFFu;  // as the codec's key_of
}

}  // namespace
}  // namespace fftsp

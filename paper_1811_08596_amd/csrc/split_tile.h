// Forward pass A with a tile in half of the LDS (fft.hip), for every kernel that works on such tiles.
#pragma once
#include "fft_core.h"

#include <type_traits>

namespace fftsp {
namespace {

constexpr int kTileFA = 13;
constexpr int tile_lanes(int loge) { return 1 << (loge - 4); }
constexpr int log_columns(int logM) { return (logM + 1) / 2; }  // log2 N1
__host__ __device__ __forceinline__ uint32_t power_tiles(int logM, int loge) { return 1u << (logM - loge); }

// Forward pass A with a tile in half of the LDS: 16 points a lane stay in registers, and between the stages real and imaginary parts go
// through LDS one after the other.  In kernels of 64 registers two tiles of 2^14 points or four of 2^13 are on a compute unit, all 32 waves of it, so
// columns of 2^11 are read 64 bytes wide instead of 32 (chunk.hip has such tiles in a kernel of 118, one to a compute unit).  What it costs is LDS instructions of four bytes instead of eight, and the persistent kernel's loads ahead.
// The same radices, twiddles and order of operations as fwd_a_run and fwd_a_tile: the bits are the same.
// Calls in us, persistent / this, 2^22 by number of tiles of 2^14: binary32 512 120.7 / 119.7, 1024 208 / 222, 1280 242.6 / 241.8, 1536 281 / 284,
//   1920 354.8 / 348.1, 3072 582 / 578, 4224 (138 M samples) 817.7 / 759.5, kernel 330 / 264 (with reads that ask for no alignment and leave out a
//   branch 230 -> 220);  binary16 1024 176 / 187, 1280 209 / 205, 1536 246 / 242.5,
//   1920 302 / 289.  Columns of 2^10, tiles of 2^13, binary16: 512 93.7 / 97.4, 640 120.5 / 121.1, 1024 146.4 / 144.7, 1280 173.5 / 172.7, 1920 261.1 / 253.2 and
//   (2^21) 272.7 / 265.9; binary32 1920 313.7 / 317.1, and with tiles of 2^14 326.  Shorter columns: equal at best.
template <int LOGN1, int LOGE>
struct SplitTile {
    static constexpr int N1 = 1 << LOGN1, LOGT = LOGE - LOGN1, T = 1 << LOGT, NT = tile_lanes(LOGE);
    static constexpr int HP = N1 / 2, LOGHP = LOGN1 - 1;
    static constexpr size_t kLds = ((size_t)sizeof(float) << LOGE) + N1 * sizeof(float2);  // a component of the tile, and the stage twiddles
    static constexpr int RL2 = stage_radix_log(LOGN1 - 3), RL3 = LOGN1 - 3 - RL2;
    static_assert(RL3 > 0 && stage_radix_log(RL3) == RL3, "three stages");
    static_assert(NT >= HP && T >= 8 && T <= 32, "a lane stores one pair of rows, of eight columns");
    // columns of a lane's stores: first(lane) + j * STEP, with the twiddles anchored every ANCHOR of them; as fwd_a_tile has them
    static constexpr int OLD = tile_lanes(kTileFA), STEP = HP >= OLD ? 1 : OLD / HP, ANCHOR = HP > OLD ? 8 * OLD / HP : 8;
    static __device__ __forceinline__ int first_column(int tid) { return (tid >> LOGHP) * (STEP > 1 ? 1 : 8); }
    // Row i, column b between two stages.  64 lanes have all columns of 64 / T neighbouring rows, or half as many lanes with column pairs have
    // them of rows eight apart: every bank once.
    static __device__ __forceinline__ int staged(int i, int b) { return ((i ^ ((i >> 3) & (64 / T - 1))) << LOGT) + b; }
    // and on the way to the stores: 64 lanes have one column of 64 neighbouring rows
    static __device__ __forceinline__ int stored(int i, int b) { return (i << LOGT) + (b ^ ((i >> (6 - LOGT)) & (T - 1))); }
    static __device__ __forceinline__ int butterfly_of(int tid, int q) { return (tid >> LOGT) + q * (NT >> LOGT); }
    template <int RL>
    static __device__ __forceinline__ int input(int tid, int n)
    {
        return staged(butterfly_of(tid, n >> RL) + (n & ((1 << RL) - 1)) * (N1 >> RL), tid & (T - 1));
    }
    template <int NS_LOG, int RL>
    static __device__ __forceinline__ int output_row(int tid, int n)
    {
        const int j = butterfly_of(tid, n >> RL);
        return ((j >> NS_LOG) << (NS_LOG + RL)) + (j & ((1 << NS_LOG) - 1)) + ((n & ((1 << RL) - 1)) << NS_LOG);
    }
    template <int NS_LOG, int RL>
    static __device__ __forceinline__ void stage(float2 (&v)[16], const float2* tw, int tid)
    {
        constexpr int RHO = 1 << RL;
#pragma unroll
        for (int q = 0; q < 16 / RHO; ++q) {
            const int k = butterfly_of(tid, q) & ((1 << NS_LOG) - 1);
#pragma unroll
            for (int t = 1; t < RHO; ++t) v[q * RHO + t] = cmul(v[q * RHO + t], tw[(t * k) << (LOGN1 - NS_LOG - RL)]);
            butterfly<RL, false>(v + q * RHO);
        }
    }
    // put(component of point n) then, behind a barrier, from(n)
    template <typename Put, typename From>
    static __device__ __forceinline__ void exchange(const float* d, float2 (&v)[16], int tid, Put&& put, From&& from)
    {
        float x[16];
        put([&](int n) __attribute__((always_inline)) { return v[n].x; }, tid);
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 16; ++n) x[n] = d[from(n, tid)];
        __syncthreads();
        const int again = opaque_lane(tid);  // addresses are computed again for the second component: kept, they spill
        put([&](int n) __attribute__((always_inline)) { return v[n].y; }, again);
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 16; ++n) v[n] = make_float2(x[n], d[from(n, again)]);
    }
};

// Samples of a lane's two butterflies of the first stage, v[q] and v[8 + q]: rows j0 + q * N1 / 8 of two neighbouring columns.
template <int LOGN1, int LOGT>
__device__ __forceinline__ void load_columns(float2 (&v)[16], const float* __restrict__ in, const Span& sp, int logM, const Tables& tb, uint32_t col0, int tid)
{
    constexpr int N1 = 1 << LOGN1, T = 1 << LOGT;
    const uint32_t M = 1u << logM, N2 = M >> LOGN1;
    const int bp = tid & (T / 2 - 1), j0 = tid >> (LOGT - 1);
    const size_t left = sp.limit > sp.first ? sp.limit - sp.first : 0;
    const uint32_t end = left >> 2 < (size_t)(M >> 1) ? (uint32_t)(left >> 2) : M >> 1;  // pieces of four samples that are whole
    const float* src = end ? in + sp.first : reinterpret_cast<const float*>(tb.hi);
    auto piece = [&](int q) __attribute__((always_inline)) { return (uint32_t)(j0 + q * (N1 / 8)) * (N2 >> 1) + (col0 >> 1) + (uint32_t)bp; };
    Floats4 r[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) r[q] = *reinterpret_cast<const Floats4*>(src + 4 * (size_t)(piece(q) < end ? piece(q) : 0u));
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const bool there = piece(q) < end;
        v[q] = there ? make_float2(r[q][0], r[q][1]) : make_float2(0.f, 0.f);
        v[8 + q] = there ? make_float2(r[q][2], r[q][3]) : make_float2(0.f, 0.f);
    }
    if ((left & 3u) != 0 && end < M >> 1) {  // the piece that the end cuts
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (piece(q) == end) {
                const size_t gi = sp.first + 4 * (size_t)end;
                v[q] = load_pair(in, gi, sp.limit);
                v[8 + q] = load_pair(in, gi + 2, sp.limit);
            }
    }
}

// One tile, columns col0 .. of a chunk whose samples are `sp` and whose intermediate is `mid`; d: 2^LOGE words; tw: the stage twiddles, which
// other lanes may still be writing.
template <int LOGN1, int LOGE, bool HALF>
__device__ __forceinline__ void fwd_a_split(const float* __restrict__ in, const Span& sp, int logM, typename Cx<HALF>::One* __restrict__ mid,
                                            const Tables& tb, uint32_t col0, float* d, const float2* tw, int tid, float in_scale)
{
    using G = SplitTile<LOGN1, LOGE>;
    constexpr int N1 = G::N1, HP = G::HP, T = G::T;
    float2 v[16];
    load_columns<LOGN1, G::LOGT>(v, in, sp, logM, tb, col0, tid);
    bf8<false>(v);
    bf8<false>(v + 8);
    G::exchange(
        d, v, tid,
        [&](auto part, int tid) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 8; ++t) *reinterpret_cast<float2*>(d + G::staged(8 * (tid >> (G::LOGT - 1)) + t, 2 * (tid & (T / 2 - 1)))) = make_float2(part(t), part(8 + t));
        },
        [&](int n, int tid) __attribute__((always_inline)) { return G::template input<G::RL2>(tid, n); });
    G::template stage<3, G::RL2>(v, tw, tid);
    __syncthreads();
    G::exchange(
        d, v, tid,
        [&](auto part, int tid) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < 16; ++n) d[G::staged(G::template output_row<3, G::RL2>(tid, n), tid & (T - 1))] = part(n);
        },
        [&](int n, int tid) __attribute__((always_inline)) { return G::template input<G::RL3>(tid, n); });
    G::template stage<3 + G::RL2, G::RL3>(v, tw, tid);
    __syncthreads();
    const uint32_t kp = (uint32_t)tid & (HP - 1);  // pair of paired positions (2kp, 2kp+1)
    const int ka = (int)kp, kb = (int)mirror_row(kp, N1), c0 = G::first_column(tid);
    G::exchange(
        d, v, tid,
        [&](auto part, int tid) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < 16; ++n) d[G::stored(G::template output_row<3 + G::RL2, G::RL3>(tid, n), tid & (T - 1))] = part(n);
        },
        [&](int n, int tid) __attribute__((always_inline)) {
            const uint32_t kp = (uint32_t)tid & (HP - 1);
            return G::stored(n & 1 ? (int)mirror_row(kp, N1) : (int)kp, G::first_column(tid) + (n >> 1) * G::STEP);
        });
    const int sh = 22 - logM;
    const float2 ratio_a = twiddle(tb, (uint32_t)(G::STEP * ka) << sh), ratio_b = twiddle(tb, (uint32_t)(G::STEP * kb) << sh);
    typename Cx<HALF>::Two* out = reinterpret_cast<typename Cx<HALF>::Two*>(mid);
    float2 cur_a, cur_b;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t n2 = col0 + (uint32_t)(c0 + j * G::STEP);
        if (j % G::ANCHOR == 0) {
            cur_a = twiddle(tb, (n2 * (uint32_t)ka) << sh);
            cur_b = twiddle(tb, (n2 * (uint32_t)kb) << sh);
            if constexpr (HALF) {  // the variant's power-of-two factors ride on the twiddles (exact)
                cur_a = make_float2(cur_a.x * in_scale, cur_a.y * in_scale);
                cur_b = make_float2(cur_b.x * in_scale, cur_b.y * in_scale);
            }
        }
        out[n2 * (uint32_t)HP + kp] = cx_store<HALF>(join(cmul(v[2 * j], cur_a), cmul(v[2 * j + 1], cur_b)));
        cur_a = cmul(cur_a, ratio_a);
        cur_b = cmul(cur_b, ratio_b);
    }
}

// 2^TOP points of tensor x by tile_lanes(TOP) lanes, share blk: one tile, or with TOP = 14 two of columns of up to 2^10.
template <int TOP>
__device__ __forceinline__ void fwd_a_split_tensor(const LongTensor& x, uint32_t blk, const float* __restrict__ in, float2* __restrict__ mid, const Tables& tb)
{
    extern __shared__ float2 smem[];
    const int logM = x.logM;
    const Span sp = chunk_span((size_t)x.goff, x.glen, 0, 0);
    auto run = [&](auto n1) __attribute__((always_inline)) {
        constexpr int LOGN1 = decltype(n1)::value, LOGE = LOGN1 > 10 ? TOP : 13;
        using G = SplitTile<LOGN1, LOGE>;
        const uint32_t sub = LOGE < TOP ? (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / G::NT) : 0u, tile = (blk << (TOP - LOGE)) + sub;
        float2* const tw = smem + (1 << TOP) / 2;
        load_stage_twiddles<LOGN1, tile_lanes(TOP)>(tw, tb, (int)threadIdx.x);
        fwd_a_split<LOGN1, LOGE, false>(in, sp, logM, mid + long_mid(x), tb, tile << G::LOGT, reinterpret_cast<float*>(smem) + (sub << LOGE), tw,
                                        (int)threadIdx.x & (G::NT - 1), 1.0f);
    };
    const int columns = log_columns(logM);
    if (columns == 8) return run(std::integral_constant<int, 8>{});
    if (columns == 9) return run(std::integral_constant<int, 9>{});
    if (TOP == 13 || columns == 10) return run(std::integral_constant<int, 10>{});
    if constexpr (TOP == 14) run(std::integral_constant<int, 11>{});
}

}  // namespace
}  // namespace fftsp

// Batched real FFT / inverse real FFT of power-of-two chunks for gfx950.
//
// The transform is the DFT sum of arXiv 1811.08596 Sec. 3.1.1 (sign -, unnormalised)
// applied per chunk, and its inverse (1/L) on the receiver (Sec. 3.1, last paragraph).
//
// Method (ours; the paper calls a vendor FFT): a real chunk of length L is read as
// M = L/2 complex samples z[j] = x[2j] + i x[2j+1]; an M-point complex FFT is followed
// by the even/odd split X[k] = E[k] + W_L^k O[k].  The M-point FFT is a Stockham
// autosort FFT held entirely in LDS (radix 8/4/2 register butterflies, one LDS
// round trip per stage).  M <= 2^14 fits one workgroup (chunk.hip, which keeps the rest of
// the codec there too).  Larger M is factored M = N1*N2 and done in two LDS-resident
// passes with a transposed intermediate (this file):
//   pass A: for a tile of TA adjacent columns n2, N1-point FFTs over n1 (stride N2),
//           times W_M^(n2 k1), stored as runs of N1 values per n2 (row k1 next to row N1-k1);
//   pass B: for a tile of rows k1 together with the mirrored rows N1-k1, N2-point
//           FFTs over n2; Z[k1 + N1 k2] and its partner Z[M-k] then sit in the same
//           workgroup, so the real-FFT split happens in LDS before the only store.
// The inverse runs the same two passes backwards (split first, 1/L at the end).
//
// LDS layout: element (i, b) of a batch of T transforms lives at i*T + (b ^ sw(i)),
// an XOR swizzle that keeps both "b fastest" and "i fastest" wave accesses spread
// over all banks without padding.
#include "fft_core.h"
#include "split_tile.h"
#include "codec_core.h"
#include "short.h"
#include <type_traits>

namespace fftsp {
namespace {

// Complex points of a tile (a power of two; 16 per lane).  A tile of 2^13 is 64 KiB of LDS, two workgroups of 512 lanes per
// compute unit.  A tile of 2^14 has a workgroup of 1024 lanes and the compute unit to itself; it is taken where the smaller
// one would touch memory in pieces of less than a 128-byte line, and there are enough of them.  Whole calls in us, small / large
// tiles in the pass, by number of the latter; nothing of a call in the caches when it starts (with everything there the lines of
// the inverse passes lie higher):
//   forward second pass, rows of 2^10 (64 -> 128 bytes), sender: 64 58.4 / 57.4, 128 67.0 / 66.1, 256 84.5 / 81.6, 1024 219 / 200,
//     4224 (138 M samples in chunks of 2^22) 913 / 810;
//   inverse second pass, the same rows, receiver: 384 80 / 84, 640 115 / 122, 1024 171 / 169 and (chunks of 2^22) 186 / 190, 1280
//     222 / 202, 4224 780 / 694; four senders' streams 1216 242 / 221;
//   inverse first pass, columns of 2^11 (stores of 32 -> 64 bytes): 128 52.1 / 52.7, 256 68.4 / 67.5, 768 157 / 146.  (Tiles in half of the
//     LDS: below.)
// With rows of 2^9, already a line wide, the second passes lose (101 / 106 and 109 / 127 us).  The forward first pass, which only
// reads in narrow pieces, was slower that way (columns of 2^10: 119 / 124 us; of 2^11: 340 us against 327 with four
// 2^13-point tiles of a line walked in step).  Binary16 storage: the same lines within 3 us.
constexpr int kWideMin = 10;  // rows (second passes) of at least 2^kWideMin
constexpr size_t kWideForward = 128, kWideInverseB = 1152;  // large tiles from which a pass takes them
constexpr size_t kWideInverseA = 256;  // columns of 2^11
inline size_t wide_tiles(size_t C, int logM) { return C << (logM - 14); }
constexpr int kLanePairs = 8;  // pairs of adjacent points a lane holds
// a pass A tile is 2^(loge - LOGN1) columns of 8 bytes; the tiles of a 128-byte line (two at least) are walked in step
constexpr int group_log(int loge, int logn1) { return loge - logn1 >= 3 ? 1 : 2; }

// The next tile's loads are issued in at most this many portions: one before the LDS stages, one after each of the
// first stages.  A wave that issues a whole tile's loads at once stands in the issue until the memory pipeline has
// taken them; in portions the stages in between proceed meanwhile.
constexpr int kSpreadA = 2;   // forward pass A (measured: 144 us whole, 137-138 in two portions, 138-141 in three)
constexpr int kSpreadFB = 3;  // forward pass B (110-112 us -> 108-109)
constexpr int kSpreadIB = 2;  // inverse pass B (114-116 -> 113)
constexpr int kSpreadIA = 3;  // inverse pass A (117 -> 115-116)
template <int LDS_LEVELS, int MOST>
constexpr int portions()
{
    return lds_stages(LDS_LEVELS) + 1 < MOST ? lds_stages(LDS_LEVELS) + 1 : MOST;
}
template <int LOGN1>
constexpr int spread_parts()
{
    return portions<LOGN1 - 3, kSpreadA>();
}

// Software pipeline of the persistent two-pass kernels.  Vector-memory results return in issue order and are
// counted by a single counter, so the order of issue decides what a wait really waits for.  Per tile t:
//     [table lookups for tile t's store loop, lookups for tile t+1's split, loads of tile t+1]   one batch
//     LDS FFT of tile t
//     store loop of tile t
//     barrier, LDS fill from the registers that hold tile t+1, barrier
// Every load is older than the stores issued after it, so no wait for a load ever waits for a store to be
// acknowledged.  The loads of the batch are unconditional (on the last tile they read one valid dummy address),
// which keeps the code between issue and use free of branches that would make the waits conservative.

// Column-to-column ratios of pass A's twiddles W_M^(n2 k1) for the row pairs a lane stores: they depend on the lane
// alone, so a workgroup looks them up once for all its tiles.
template <int LOGN1>
struct PassARatios {
    static constexpr int NT = tile_lanes(kTileFA), HP = (1 << LOGN1) / 2;
    static constexpr int KN = HP >= NT ? HP / NT : 1;
    float2 a[KN], b[KN];
};
template <int LOGN1>
__device__ __forceinline__ PassARatios<LOGN1> pass_a_ratios(const Tables& tb, int logM, int tid)
{
    constexpr int N1 = 1 << LOGN1, HP = N1 / 2, KN = PassARatios<LOGN1>::KN, NT = PassARatios<LOGN1>::NT;
    constexpr int DC = HP >= NT ? 1 : NT / HP;
    PassARatios<LOGN1> r;
#pragma unroll
    for (int kk = 0; kk < KN; ++kk) {
        const uint32_t kp = (uint32_t)(tid + kk * NT) & (HP - 1);
        r.a[kk] = twiddle(tb, ((uint32_t)DC * kp) << (22 - logM));
        r.b[kk] = twiddle(tb, ((uint32_t)DC * mirror_row(kp, N1)) << (22 - logM));
    }
    return r;
}

// One tile of pass A once its first stage is in LDS: the twiddle look-ups of the store loop, `prefetch()` (loads of
// a later tile, issued here so that they are older than this tile's stores), the LDS stages, and the store loop,
// which multiplies by W_M^(n2 k1) and writes row k1 next to row N1 - k1.
template <int LOGN1, bool HALF, typename Prefetch>
__device__ __forceinline__ void fwd_a_tile(uint32_t t, uint32_t tiles, int logM, typename Cx<HALF>::One* __restrict__ mid,
                                           const Tables& tb, float2* d, const float2* tw, int tid, float in_scale,
                                           const PassARatios<LOGN1>& ratio, Prefetch prefetch)
{
    constexpr int LOGE = kTileFA, NT = tile_lanes(LOGE), PER2 = kLanePairs;
    constexpr int N1 = 1 << LOGN1, LOGT = LOGE - LOGN1;
    constexpr int HP = N1 / 2, LOGHP = LOGN1 - 1;  // row pairs per column
    constexpr int KN = HP >= NT ? HP / NT : 1;   // distinct row pairs per lane in the store loop
    constexpr int DC = HP >= NT ? 1 : NT / HP;   // column step between a lane's consecutive stores
    constexpr int NCOL = PER2 / KN;
    static_assert(NCOL <= 8, "twiddle recurrence is anchored once");
    const uint32_t M = 1u << logM;
    const uint32_t col0 = tile_in_chunk(t, tiles) << LOGT;
    const int sh = 22 - logM;
    float2 cur_a[KN], cur_b[KN];
#pragma unroll
    for (int kk = 0; kk < KN; ++kk) {
        const uint32_t kp = (uint32_t)(tid + kk * NT) & (HP - 1);
        const uint32_t ka = kp, kb = mirror_row(kp, N1);
        const uint32_t cfirst = (uint32_t)(tid + kk * NT) >> LOGHP;
        cur_a[kk] = twiddle(tb, ((col0 + cfirst) * ka) << sh);
        cur_b[kk] = twiddle(tb, ((col0 + cfirst) * kb) << sh);
        if constexpr (HALF) {  // the variant's power-of-two factors ride on the twiddles (exact)
            cur_a[kk] = make_float2(cur_a[kk].x * in_scale, cur_a[kk].y * in_scale);
            cur_b[kk] = make_float2(cur_b[kk].x * in_scale, cur_b[kk].y * in_scale);
        }
    }
    // the next tile's loads go out in kSpreadA portions: one before the LDS stages, one after each of the first stages
    prefetch(0);
    run_fft_between<LOGN1, LOGT, NT, false, 3>(d, tw, tid, [&](int k) {
        if (k + 1 < spread_parts<LOGN1>()) prefetch(k + 1);
    });
    typename Cx<HALF>::Two* out = reinterpret_cast<typename Cx<HALF>::Two*>(mid + (size_t)(t / tiles) * (size_t)M);
#pragma unroll
    for (int kk = 0; kk < KN; ++kk) {
        const uint32_t kp = (uint32_t)(tid + kk * NT) & (HP - 1);  // pair of paired positions (2kp, 2kp+1)
        const uint32_t ka = kp, kb = mirror_row(kp, N1);
        const uint32_t cfirst = (uint32_t)(tid + kk * NT) >> LOGHP;
#pragma unroll
        for (int j = 0; j < NCOL; ++j) {
            const uint32_t col = cfirst + j * DC, n2 = col0 + col;
            const float2 va = cmul(d[sw_idx<LOGT>((int)ka, (int)col)], cur_a[kk]);
            const float2 vb = cmul(d[sw_idx<LOGT>((int)kb, (int)col)], cur_b[kk]);
            out[n2 * (uint32_t)HP + kp] = cx_store<HALF>(join(va, vb));
            cur_a[kk] = cmul(cur_a[kk], ratio.a[kk]);
            cur_b[kk] = cmul(cur_b[kk], ratio.b[kk]);
        }
    }
}

// Forward pass A: N1-point FFTs down the columns of the N1 x N2 view of z, for tiles of TA adjacent columns.
// kWhole: every tile of this workgroup's run lies in a chunk that is wholly inside the input, and the input is
// 16-byte aligned: two columns per 16-byte load, no guards.  kGuarded: every element is loaded under a guard (ragged ends).
// The variants are separate loops so that no branches stand between the unguarded ones' loads and their use.
enum Reads { kGuarded, kWhole };
template <int LOGN1, Reads MODE, bool HALF>
__device__ __forceinline__ void fwd_a_run(const float* __restrict__ in, size_t n, int logM,
                                          typename Cx<HALF>::One* __restrict__ mid, const Tables& tb, uint32_t t, uint32_t tend, uint32_t tstep, float2* d, const float2* tw, int tid0,
                                          float in_scale)
{
    constexpr int LOGE = kTileFA, NT = tile_lanes(LOGE), PER2 = kLanePairs;
    constexpr int N1 = 1 << LOGN1, LOGT = LOGE - LOGN1, TA = 1 << LOGT;
    static_assert(LOGT >= 2 && (NT % (TA / 2)) == 0, "tile shape");
    const uint32_t M = 1u << logM, N2 = M >> LOGN1, tiles = N2 >> LOGT;

    // live = false: the tile does not exist; the fast loads are still issued, all to one valid address
    // part p of spread_parts(): loads q with q * parts / PER2 == p; prologue calls pass every part in turn
    auto load_tile = [&](float4 (&r)[PER2], uint32_t tile, int tid, bool live, int part) {
        // every tile lies in a real chunk, so the span needs no chunk count
        const Span sp = chunk_span(0, n, tile / tiles, 2 * (size_t)M);
        const uint32_t col0 = tile_in_chunk(tile, tiles) << LOGT;
        if constexpr (MODE == kWhole) {
            const float4* src = live ? reinterpret_cast<const float4*>(in + sp.first) + (col0 >> 1)
                                     : reinterpret_cast<const float4*>(tb.hi);
#pragma unroll
            for (int q = 0; q < PER2; ++q) {
                if (q * spread_parts<LOGN1>() / PER2 != part) continue;
                const int w = tid + q * NT, bp = w & (TA / 2 - 1), n1 = w >> (LOGT - 1);
                r[q] = src[live ? (uint32_t)n1 * (N2 >> 1) + bp : 0u];
            }
        } else {
            if (!live || part != 0) return;
#pragma unroll
            for (int q = 0; q < PER2; ++q) {
                const int w = tid + q * NT, bp = w & (TA / 2 - 1), n1 = w >> (LOGT - 1);
                const size_t gi = sp.first + 2 * ((size_t)n1 * N2 + col0 + 2 * bp);
                r[q] = join(load_pair(in, gi, sp.limit), load_pair(in, gi + 2, sp.limit));
            }
        }
    };
    // r[q] holds rows (tid >> (LOGT-1)) + q * N1/8 of one column pair: the first stage runs on the way into LDS
    static_assert(PER2 == 8 && (NT >> (LOGT - 1)) == N1 / 8, "a lane's loads are the inputs of two radix-8 butterflies");
    auto fill = [&](float4 (&r)[PER2], uint32_t tile, int tid) {
        first_stage_store<LOGT, false>(d, tid >> (LOGT - 1), 2 * (tid & (TA / 2 - 1)), r);
    };
    float4 r[PER2];
#pragma unroll
    for (int part = 0; part < spread_parts<LOGN1>(); ++part) load_tile(r, t, tid0, true, part);
    const PassARatios<LOGN1> ratio = pass_a_ratios<LOGN1>(tb, logM, tid0);
    fill(r, t, tid0);
    __syncthreads();
    for (;;) {
        const int tid = opaque_lane(tid0);
        const bool more = t + tstep < tend;
        fwd_a_tile<LOGN1, HALF>(t, tiles, logM, mid, tb, d, tw, tid, in_scale, ratio,
                                [&](int part) { load_tile(r, more ? t + tstep : t, tid, more, part); });
        if (!more) break;
        t += tstep;
        __syncthreads();
        fill(r, t, tid);
        __syncthreads();
    }
}

// The tiles of workgroup blk of a pass A over the chunks of in[0 .. n), in chunks of 2^(logM+1).
// `aligned`: `in` is 16-byte aligned.
template <int LOGN1, bool HALF>
__device__ __forceinline__ void fwd_a_workgroup(uint32_t blk, const float* __restrict__ in, size_t n, int logM,
                                                typename Cx<HALF>::One* __restrict__ mid, const Tables& tb, bool aligned,
                                                uint32_t total, uint32_t per_wg, int glog, float in_scale)
{
    constexpr int LOGE = kTileFA, NT = tile_lanes(LOGE), ELEMS = 1 << LOGE;
    extern __shared__ float2 smem[];
    float2* d = smem;
    float2* tw = smem + ELEMS;
    const int tid0 = threadIdx.x;
    uint32_t t, tend;
    if (!grouped_run(blk, total, per_wg, glog, t, tend)) return;
    load_stage_twiddles<LOGN1, NT>(tw, tb, tid0);
    const uint32_t tiles = (1u << logM) >> LOGE;  // tiles per chunk
    const size_t last_chunk_end = ((size_t)((tend - 1) / tiles) + 1) << (logM + 1);
    if (aligned && last_chunk_end <= n)
        fwd_a_run<LOGN1, kWhole, HALF>(in, n, logM, mid, tb, t, tend, 1u << glog, d, tw, tid0, in_scale);
    else
        fwd_a_run<LOGN1, kGuarded, HALF>(in, n, logM, mid, tb, t, tend, 1u << glog, d, tw, tid0, in_scale);
}

template <int LOGN1, bool HALF>
__global__ __launch_bounds__(tile_lanes(kTileFA)) void k_fwd_a(const float* __restrict__ in, size_t n, int logM,
                                               typename Cx<HALF>::One* __restrict__ mid, Tables tb, bool aligned,
                                               uint32_t total, uint32_t per_wg, int glog, uint32_t* __restrict__ zero_ptr,
                                               uint32_t zero_words, float in_scale, const uint32_t* __restrict__ only_if)
{
    constexpr int NT = tile_lanes(kTileFA);
    if (only_if && *only_if == 0u) return;  // stand-by launch behind a fused kernel that did finish
    // clears the status words and key histograms the next kernels of the sender accumulate into
    for (uint32_t i = blockIdx.x * NT + threadIdx.x; i < zero_words; i += gridDim.x * NT) zero_ptr[i] = 0u;
    fwd_a_workgroup<LOGN1, HALF>(blockIdx.x, in, n, logM, mid, tb, aligned, total, per_wg, glog, in_scale);
}

// The tiles of a few tensors, 2^13 points to a workgroup of their own, whole in the LDS: two to a compute unit and half as many trips through it as in
// half of it.  Figures at whole_forward.
__global__ __launch_bounds__(tile_lanes(kTileFA)) void k_fwd_a_long(const float* __restrict__ in, float2* __restrict__ mid, Tables tb, uint32_t total, uint32_t step,
                                                                   uint32_t* __restrict__ zero_ptr, uint32_t zero_words, LongTable tab, LongStarts at)
{
    constexpr int LOGE = kTileFA, NT = tile_lanes(LOGE);
    extern __shared__ float2 smem[];
    float2 *const d = smem, *const tw = smem + (1 << LOGE);
    for (uint32_t i = blockIdx.x * NT + threadIdx.x; i < zero_words; i += gridDim.x * NT) zero_ptr[i] = 0u;
    const uint32_t t = in_turned_stretches(total, step);
    if (t >= total) return;
    const LongShare share = long_share(at, t);
    const LongTensor& x = tab.t[share.tensor];
    const int logM = x.logM, tid = threadIdx.x;
    auto run = [&](auto n1) __attribute__((always_inline)) {
        constexpr int LOGN1 = decltype(n1)::value, LOGT = LOGE - LOGN1;
        load_stage_twiddles<LOGN1, NT>(tw, tb, tid);
        float2 v[16];
        load_columns<LOGN1, LOGT>(v, in, chunk_span((size_t)x.goff, x.glen, 0, 0), logM, tb, share.blk << LOGT, tid);
        const PassARatios<LOGN1> ratio = pass_a_ratios<LOGN1>(tb, logM, tid);
        float4 r[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = join(v[q], v[8 + q]);
        first_stage_store<LOGT, false>(d, tid >> (LOGT - 1), 2 * (tid & ((1 << LOGT) / 2 - 1)), r);
        __syncthreads();
        fwd_a_tile<LOGN1, false>(share.blk, power_tiles(logM, LOGE), logM, mid + long_mid(x), tb, d, tw, tid, 1.0f, ratio, [](int) {});
    };
    switch (log_columns(logM)) {
        case 8: return run(std::integral_constant<int, 8>{});
        case 9: return run(std::integral_constant<int, 9>{});
        case 10: return run(std::integral_constant<int, 10>{});
        default: return run(std::integral_constant<int, 11>{});
    }
}


// From how many tiles of 2^14, columns of 2^11, forward pass A has them in half of the LDS (split_tile.h); figures there.
template <bool HALF>
constexpr size_t kSplitForward = HALF ? 1280 : 1792;  // tiles of 2^14, columns of 2^11
template <int LOGN1, int LOGE, bool HALF>
__global__ __launch_bounds__(tile_lanes(LOGE)) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_fwd_a_split(
    const float* __restrict__ in, size_t n, int logM, typename Cx<HALF>::One* __restrict__ mid, Tables tb, uint32_t total,
    uint32_t* __restrict__ zero_ptr, uint32_t zero_words, float in_scale)
{
    using G = SplitTile<LOGN1, LOGE>;
    extern __shared__ float2 smem[];
    float* const d = reinterpret_cast<float*>(smem);
    float2* const tw = smem + (1 << LOGE) / 2;
    const int tid = threadIdx.x;
    // clears the status words and key histograms the next kernels of the sender accumulate into
    for (uint32_t i = blockIdx.x * G::NT + tid; i < zero_words; i += gridDim.x * G::NT) zero_ptr[i] = 0u;
    const uint32_t t = in_stretches(total);
    if (t >= total) return;
    const int log_tiles = logM - LOGE;
    const uint32_t c = t >> log_tiles;
    const Span sp = chunk_span(0, n, c, (size_t)2 << logM);
    load_stage_twiddles<LOGN1, G::NT>(tw, tb, tid);
    fwd_a_split<LOGN1, LOGE, HALF>(in, sp, logM, mid + ((size_t)c << logM), tb, (t & ((1u << log_tiles) - 1u)) << G::LOGT, d, tw, tid, in_scale);
}

// Forward pass B: N2-point FFTs along n2 for a tile of rows and their mirrors, then the real-FFT split.
// A lane owns one pair of slots (row ka and its mirror kb), i.e. 16 bytes of every run it touches.
// CODEC: the spectrum is stored in the paired order and the first radix-select digit of every bin's key is
// counted into the 12-bit histogram of the chunk (hist); otherwise natural bin order and no histogram.
// The store loop is free of branches (partner addresses and the rare self-mirrored rows are handled with
// selects) so that its LDS reads can be issued ahead in batches instead of one wait per read.
// HALF (CODEC only): the intermediate is read and the spectrum written as binary16 pairs; the histogram counts
// the keys of the values as stored, which are the ones the selection will see.
// Workgroup blk of nblk does its share of the total tiles.
template <int LOGN2, int LOGE, bool CODEC, bool HALF>
__device__ __forceinline__ void fwd_b_workgroup(uint32_t blk, uint32_t nblk, const typename Cx<HALF>::One* __restrict__ mid,
                                                int logM, typename Cx<HALF>::One* __restrict__ spec, uint32_t sstride,
                                                const Tables& tb, uint32_t* __restrict__ hist, uint32_t total,
                                                uint32_t per_wg, float mid_scale)
{
    static_assert(CODEC || !HALF, "binary16 storage is the codec's own");
    using Two = typename Cx<HALF>::Two;
    constexpr int NT = tile_lanes(LOGE), PER2 = kLanePairs;
    constexpr int N2 = 1 << LOGN2, LOGT = LOGE - LOGN2, ELEMS = 1 << LOGE;
    constexpr int LOGP = LOGT - 1, P = 1 << LOGP;  // slot pairs per tile
    static_assert(LOGT >= 1 && NT % P == 0, "a lane keeps one slot pair");
    extern __shared__ float2 smem[];
    float2* d = smem;
    float2* tw = smem + ELEMS;
    uint32_t* h16 = reinterpret_cast<uint32_t*>(tw + N2);
    const int tid0 = threadIdx.x;
    const int logN1 = logM - LOGN2;
    const uint32_t M = 1u << logM, N1 = 1u << logN1, tiles = N1 >> LOGT;
    // runs differ by at most one tile: the first total - per_wg * nblk workgroups take one more
    const uint32_t extra = total - per_wg * nblk;
    uint32_t t = blk * per_wg + (blk < extra ? blk : extra);
    const uint32_t tend = t + per_wg + (blk < extra ? 1u : 0u);
    if (t >= tend) return;
    load_stage_twiddles<LOGN2, NT>(tw, tb, tid0);
    if (CODEC)
        for (int i = tid0; i < kHistLdsWords; i += NT) h16[i] = 0u;
    constexpr int DK = NT >> LOGP;  // k2 step between a lane's consecutive pairs
    static_assert(2 * kSplitStep * (PER2 - 1) < 16, "split twiddle steps stay inside the 32nd-root table");
    // the LDS histogram has 16-bit counters and a tile adds at most 2^LOGE + 1 keys
    constexpr uint32_t kFlushEvery = 65535u / ((1u << LOGE) + 1u);
    static_assert(LOGE != 13 || kFlushEvery == 7, "flush after at most 7 tiles");
    constexpr int BATCH = 4;  // pairs whose LDS reads are issued together
    static_assert(PER2 % BATCH == 0, "batches divide the store loop");

    Two r[PER2];
    constexpr int PARTS = portions<LOGN2 - 3, kSpreadFB>();
    // part < 0: the whole tile; otherwise the loads q with q * PARTS / PER2 == part
    auto load_tile = [&](uint32_t tile, int tid, bool live, int part = -1) {
        const int p = tid & (P - 1), kq0 = tid >> LOGP;
        const Two* src = reinterpret_cast<const Two*>(mid + (live ? (size_t)(tile / tiles) * (size_t)M : 0));
        const uint32_t pp = tile_in_chunk(tile, tiles) * P + p;
#pragma unroll
        for (int q = 0; q < PER2; ++q)
            if (part < 0 || q * PARTS / PER2 == part) r[q] = src[live ? (uint32_t)(kq0 + q * DK) * (N1 >> 1) + pp : 0u];
    };
    // r[q] holds rows kq0 + q * N2/8 of one slot pair: the first radix-8 stage runs on the way into LDS
    static_assert(PER2 == 8 && DK == N2 / 8, "a lane's loads are the inputs of two radix-8 butterflies");
    auto fill = [&](int tid) {
        const int p = tid & (P - 1), kq0 = tid >> LOGP;
        float4 v[PER2];
#pragma unroll
        for (int q = 0; q < PER2; ++q) v[q] = cx_load(r[q]);
        first_stage_store<LOGT, false>(d, kq0, 2 * p, v);
    };
    // the factor that kept the stored intermediate inside binary16's range is undone in the split (a power of two: exact)
    const float unlift = HALF ? mid_scale : 1.f, half = 0.5f * unlift;
    // one key into the 16-bit LDS histogram (bucket b: word b/2, half b%2); on = false adds nothing
    auto count = [&](float2 x, bool on) {
        const uint32_t b = fft_key_of(x) >> kKeyShift;
        atomicAdd(&h16[b >> 1], on ? 1u << ((b & 1u) * 16u) : 0u);
    };
    load_tile(t, tid0, true);
    fill(tid0);
    __syncthreads();
    uint32_t unflushed = 0;
    for (;;) {
        const int tid = opaque_lane(tid0);
        const int p = tid & (P - 1), kq0 = tid >> LOGP;
        const uint32_t pp = tile_in_chunk(t, tiles) * P + p;
        const uint32_t ka = pp, kb = mirror_row(pp, N1);
        const bool self = pp == 0;  // rows 0 and N1/2 are their own mirrors
        // W_L^(k1 + N1*k2): k2 advances by DK per step, i.e. by exactly 2*kSplitStep 32nds of a turn
        const float2 base_a = twiddle(tb, (ka + ((uint32_t)kq0 << logN1)) << (21 - logM));
        const float2 base_b = twiddle(tb, (kb + ((uint32_t)kq0 << logN1)) << (21 - logM));
        const bool more = t + 1 < tend;
        load_tile(more ? t + 1 : t, tid, more, 0);
        run_fft_between<LOGN2, LOGT, NT, false, 3>(d, tw, tid, [&](int k) {
            if (k + 1 < PARTS) load_tile(more ? t + 1 : t, tid, more, k + 1);
        });
        const size_t c = t / tiles;
        typename Cx<HALF>::One* out = spec + c * (size_t)sstride;
#pragma unroll
        for (int q0 = 0; q0 < PER2; q0 += BATCH) {
            float2 a0[BATCH], a1[BATCH], pa[BATCH], pb[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int k2 = kq0 + (q0 + u) * DK, k2p = N2 - 1 - k2;
                // X[ka, k2] pairs with Z[kb, N2-1-k2] and X[kb, k2] with Z[ka, N2-1-k2]; row 0 pairs with itself
                // at (N2-k2) mod N2 and row N1/2 with itself at N2-1-k2
                const int ia = self ? sw_idx<LOGT>((N2 - k2) & (N2 - 1), 2 * p) : sw_idx<LOGT>(k2p, 2 * p + 1);
                const int ib = self ? sw_idx<LOGT>(k2p, 2 * p + 1) : sw_idx<LOGT>(k2p, 2 * p);
                a0[u] = d[sw_idx<LOGT>(k2, 2 * p)];
                a1[u] = d[sw_idx<LOGT>(k2, 2 * p + 1)];
                pa[u] = d[ia];
                pb[u] = d[ib];
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int q = q0 + u, k2 = kq0 + q * DK;
                const float2 wq = make_float2(kW32re[2 * q * kSplitStep], kW32im[2 * q * kSplitStep]);
                float2 xa = split_fwd(a0[u], pa[u], cmul(base_a, wq), half);
                const float2 xb = split_fwd(a1[u], pb[u], cmul(base_b, wq), half);
                if (q == 0) {  // k2 = 0 only here: bin 0 and the Nyquist bin come from Z[0] alone
                    const bool dc = self && kq0 == 0;
                    const typename Cx<HALF>::One xm_st = cx_store<HALF>(make_float2((a0[u].x - a0[u].y) * unlift, 0.f));
                    if (dc) {
                        xa = make_float2((a0[u].x + a0[u].y) * unlift, 0.f);
                        out[M] = xm_st;
                    }
                    if (CODEC) count(cx_load(xm_st), dc);
                }
                if constexpr (CODEC) {
                    const Two st = cx_store<HALF>(join(xa, xb));
                    reinterpret_cast<Two*>(out)[((uint32_t)k2 << (logN1 - 1)) + pp] = st;
                    const float4 seen = cx_load(st);  // what the selection will read back
                    count(lo2(seen), true);
                    count(hi2(seen), true);
                } else {
                    out[ka + ((uint32_t)k2 << logN1)] = xa;
                    out[kb + ((uint32_t)k2 << logN1)] = xb;
                }
            }
        }
        ++unflushed;
        if (CODEC && (!more || unflushed == kFlushEvery || (t + 1) / tiles != c)) {
            __syncthreads();
            uint32_t* g = hist + c * kHistBins;
            // neighbouring lanes add to neighbouring counters: where a workgroup has few tiles, the flush is its tail (a tile of 2^14
            // each: ResNet-50's longest tensors 34.7 -> 32.2 us)
            for (int i = tid; i < 2 * kHistLdsWords; i += NT) {
                const uint32_t v = h16[i >> 1] >> (16 * (i & 1)) & 0xFFFFu;
                if (v) {
                    atomicAdd(&g[i], v);
                    h16[i >> 1] = 0u;  // the wave has read both halves
                }
            }
            unflushed = 0;
        }
        if (!more) break;
        ++t;
        __syncthreads();
        fill(tid);
        __syncthreads();
    }
}

template <int LOGN2, int LOGE, bool CODEC, bool HALF>
__global__ __launch_bounds__(tile_lanes(LOGE)) void k_fwd_b(const typename Cx<HALF>::One* __restrict__ mid, int logM,
                                               typename Cx<HALF>::One* __restrict__ spec, uint32_t sstride, Tables tb,
                                               uint32_t* __restrict__ hist, uint32_t total, uint32_t per_wg,
                                               float mid_scale, const uint32_t* __restrict__ only_if)
{
    if (only_if && *only_if == 0u) return;  // stand-by launch behind a fused kernel that did finish
    fwd_b_workgroup<LOGN2, LOGE, CODEC, HALF>(blockIdx.x, gridDim.x, mid, logM, spec, sstride, tb, hist, total, per_wg, mid_scale);
}

// The same for the codec with a tile in half of the LDS (HalfTile), one to a workgroup: eight pairs of rows from pp0 on.
//
// The last stage leaves a lane rows that are each other's mirrors, so the split needs no trip through LDS; lanes 32 apart have each
// other's mirrored rows, and swap, so that a lane stores pairs.
//
// Bound by the two trips to memory that nothing hides but the other workgroups of the compute unit, and by the stages.  Binary16, 62 M samples in
// chunks of 2^20: 80 us for 50 of traffic (99 as fwd_b_workgroup).  Six waves a SIMD, two registers spilled: eight spill twenty (125 us), and the
// histogram in the tile's place, which they would need, costs two barriers and 11 us with six.  Runs of tiles that share a
// histogram spill, too (115).  Rows of 2^10 are workgroups of sixteen waves, so it is four waves a SIMD or eight; eight spill twenty registers, and two
// workgroups beside each other are worth it: senders, four / eight, 2^21 17 M 120.2 / 113.1, 62 M 294.5 / 270.1; 2^22 62 M 323.0 / 292.4 (fwd_b_workgroup 116.8, 287.3, 324.7).
// With eight, the split's twiddles looked up before the stages / behind them, when registers are free again: 2^21 40 M 192.1 / 186.9, 62 M 267.7 / 259.7; 2^22 62 M 293.7 / 284.6.
__device__ __forceinline__ void swap_halves(uint32_t& a, uint32_t& b)  // lanes 32 .. 63 of a with lanes 0 .. 31 of b
{
    const auto v = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = v[0];
    b = v[1];
}
__device__ __forceinline__ void swap_halves(float2& a, float2& b)
{
    uint32_t ax = __float_as_uint(a.x), ay = __float_as_uint(a.y), bx = __float_as_uint(b.x), by = __float_as_uint(b.y);
    swap_halves(ax, bx);
    swap_halves(ay, by);
    a = make_float2(__uint_as_float(ax), __uint_as_float(ay));
    b = make_float2(__uint_as_float(bx), __uint_as_float(by));
}
__device__ __forceinline__ float4 two_of(float2 a, float2 b) { return join(a, b); }
__device__ __forceinline__ uint2 two_of(uint32_t a, uint32_t b) { return make_uint2(a, b); }
template <int LOGN2, bool HALF, int TOP = LOGN2>
__device__ __forceinline__ void fwd_b_pairs(const typename Cx<HALF>::One* __restrict__ mid, int logM, typename Cx<HALF>::One* __restrict__ spec,
                                            const Tables& tb, uint32_t* __restrict__ hist, uint32_t pp0, bool first, uint32_t* lds, int lane,
                                            float mid_scale)
{
    using G = HalfTile<LOGN2>;
    using One = typename Cx<HALF>::One;
    using Two = typename Cx<HALF>::Two;
    constexpr int N2 = G::N2, NT = G::NT, DK = G::DK, P = G::PAIRS;
    // 2^(TOP - LOGN2) tiles beside each other, each with LDS of its own, share the histogram behind them
    constexpr int LANES = NT << (TOP - LOGN2);
    const int tid = lane & (NT - 1), sub = __builtin_amdgcn_readfirstlane(lane / NT);
    float* const d = reinterpret_cast<float*>(lds + sub * (int)(G::kLds / 4));
    float2* const tw = reinterpret_cast<float2*>(d + N2 * G::SLOTS);
    uint32_t* const h16 = lds + (G::kLds / 4 << (TOP - LOGN2));  // 16-bit counters: there are 2^14 + 1 keys at most
    const int logN1 = logM - LOGN2, p = tid & (P - 1), kq = tid >> 3;
    const uint32_t M = 1u << logM, N1 = 1u << logN1, pp = pp0 + (uint32_t)p;
    Two raw[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
        raw[q] = *reinterpret_cast<const Two*>(reinterpret_cast<const uint8_t*>(mid) + (((uint32_t)(kq + q * DK) << (logN1 - 1)) + pp) * (uint32_t)sizeof(Two));
    load_stage_twiddles<LOGN2, NT>(tw, tb, tid);
    for (int i = 4 * lane; i < kHistLdsWords; i += 4 * LANES) *reinterpret_cast<uint4*>(h16 + i) = make_uint4(0u, 0u, 0u, 0u);
    // a wave has four rows of a pair in its lower lanes and their mirrors in the upper ones
    const int hi = (tid >> 5) & 1, low_row = 4 * (tid >> 6) + ((tid >> 3) & 3);
    const MirroredRows<LOGN2> rows(pp, hi ? DK - 1 - low_row : low_row);
    // W_L^(k1 + N1*k2): k2 advances by N2/8 per step, i.e. by a sixteenth of a turn
    float2 base[2];
    auto split_twiddles = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            base[i] = twiddle(tb, ((rows.upper(i) ? mirror_row(pp, N1) : pp) + ((uint32_t)rows.at(i) << logN1)) << (21 - logM));
    };
    if constexpr (TOP < 10) split_twiddles();  // eight waves have no registers to hold them in meanwhile
    float2 v[16];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float4 z = cx_load(raw[q]);
        v[q] = lo2(z);
        v[8 + q] = hi2(z);
    }
    bf8<false>(v);
    bf8<false>(v + 8);
    auto row_of = [&](int q) __attribute__((always_inline)) { return G::row_of(tid, q); };
    auto mirrored = [&](int n) __attribute__((always_inline)) {
        return G::template at_row<DK>(rows.at(n >> 3), n & 7, rows.upper(n >> 3) * P + p);
    };
    G::exchange(
        d, v, [&](int n) __attribute__((always_inline)) { return G::first_output(kq, n & 7, n < 8 ? p : P + p); },
        [&](int n) __attribute__((always_inline)) { return G::template input<G::RL2>(tid, n); });
    G::template stage<false, 3, G::RL2>(v, tw, row_of);
    G::exchange(d, v, [&](int n) __attribute__((always_inline)) { return G::second_output(tid, n); }, mirrored);
    if constexpr (G::RL3 > 0) {
        static_assert(G::RL3 == 0 || G::LAST == 3, "two butterflies of eight rows");
        G::template stage<false, 3 + G::RL2, G::LAST>(v, tw, [&](int q) __attribute__((always_inline)) { return rows.at(q); });
    }
    if constexpr (TOP >= 10) split_twiddles();
    const float unlift = HALF ? mid_scale : 1.f, half = 0.5f * unlift;
    auto turned = [&](int i, int q) __attribute__((always_inline)) { return cmul(base[i], make_float2(kW32re[2 * q], kW32im[2 * q])); };
    auto count = [&](One st) __attribute__((always_inline)) {  // what the selection will read back
        const uint32_t b = fft_key_of(cx_load(st)) >> kKeyShift;
        atomicAdd(&h16[b >> 1], 1u << ((b & 1u) * 16u));
    };
    if (first) {
        auto either = [](bool which, float2 a, float2 b) __attribute__((always_inline)) { return make_float2(which ? a.x : b.x, which ? a.y : b.y); };
        auto put = [&](int i, int q, float2 x) __attribute__((always_inline)) {
            const One st = cx_store<HALF>(x);
            spec[((uint32_t)(rows.at(i) + q * DK) << logN1) + 2u * pp + (uint32_t)rows.upper(i)] = st;
            count(st);
        };
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            __builtin_amdgcn_sched_barrier(0);
            const float2 pa = either(rows.alone, v[(8 - q) & 7], v[15 - q]), pb = either(rows.alone, v[15 - q], v[7 - q]);
            float2 x = split_fwd(v[q], pa, turned(0, q), half);
            if (q == 0 && rows.alone) {  // bin 0 and the Nyquist bin come from Z[0] alone
                x = make_float2((v[0].x + v[0].y) * unlift, 0.f);
                const One last = cx_store<HALF>(make_float2((v[0].x - v[0].y) * unlift, 0.f));
                spec[M] = last;
                count(last);
            }
            put(0, q, x);
            put(1, q, split_fwd(v[8 + q], pb, turned(1, q), half));
        }
    } else {
        auto put = [&](uint32_t i, Two z) __attribute__((always_inline)) {
            *reinterpret_cast<Two*>(reinterpret_cast<uint8_t*>(spec) + i * (uint32_t)sizeof(Two)) = z;
        };
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            __builtin_amdgcn_sched_barrier(0);
            const int u = 7 - t;
            One xt = cx_store<HALF>(split_fwd(v[t], v[15 - t], turned(0, t), half)), xu = cx_store<HALF>(split_fwd(v[u], v[15 - u], turned(0, u), half));
            One yt = cx_store<HALF>(split_fwd(v[8 + t], v[u], turned(1, t), half)), yu = cx_store<HALF>(split_fwd(v[8 + u], v[t], turned(1, u), half));
            count(xt);
            count(xu);
            count(yt);
            count(yu);
            swap_halves(xt, xu);
            swap_halves(yt, yu);
            const uint32_t q = (uint32_t)(hi ? u : t) * DK;
            put((((uint32_t)low_row + q) << (logN1 - 1)) + pp, two_of(xt, yu));
            put((((uint32_t)(DK - 1 - low_row) + q) << (logN1 - 1)) + pp, two_of(xu, yt));
        }
    }
    __syncthreads();
    // two counters at a time: neither carries into the other
    for (int i = lane; i < kHistLdsWords; i += LANES) {
        const uint32_t n = h16[i];
        if (n) atomicAdd(reinterpret_cast<unsigned long long*>(hist) + i, (unsigned long long)(n >> 16) << 32 | (n & 0xFFFFu));
    }
}
template <int LOGN2, bool HALF>  // (rows of 2^10: a workgroup of sixteen waves)
__global__ __launch_bounds__(HalfTile<LOGN2>::NT) __attribute__((amdgpu_waves_per_eu(LOGN2 == 10 ? 8 : 6, LOGN2 == 10 ? 8 : 6))) void k_fwd_b_pairs(
    const typename Cx<HALF>::One* __restrict__ mid, int logM, typename Cx<HALF>::One* __restrict__ spec, uint32_t sstride, Tables tb,
    uint32_t* __restrict__ hist, uint32_t total, float mid_scale)
{
    extern __shared__ float2 smem[];
    const int log_tiles = logM - LOGN2 - 4;
    const uint32_t t = in_stretches(total);
    if (t >= total) return;
    const uint32_t c = t >> log_tiles, pp0 = (t & ((1u << log_tiles) - 1u)) * HalfTile<LOGN2>::PAIRS;
    fwd_b_pairs<LOGN2, HALF>(mid + ((size_t)c << logM), logM, spec + c * (size_t)sstride, tb, hist + (size_t)c * kHistBins, pp0, pp0 == 0,
                             reinterpret_cast<uint32_t*>(smem), threadIdx.x, mid_scale);
}

// Tensors of different lengths: a workgroup does one tile of rows of 2^TOP, two of half the length, four of a quarter, and so on.  Rows of 2^9 spill in
// workgroups of sixteen waves, too (see fwd_b_pairs), and those of 2^10 in any; it is fewer tails that gain.
template <int TOP>
constexpr size_t kPairsLds = HalfTile<TOP>::kLds + kHistLdsWords * sizeof(uint32_t);
template <int TOP>
__global__ __launch_bounds__(HalfTile<TOP>::NT) __attribute__((amdgpu_waves_per_eu(TOP == 10 ? 8 : 6, TOP == 10 ? 8 : 6))) void k_fwd_b_pairs_long(
    const float2* __restrict__ mid, float2* __restrict__ spec, Tables tb, uint32_t* __restrict__ hist, uint32_t total, uint32_t few, LongTable tab, LongStarts at)
{
    extern __shared__ float2 smem[];
    const uint32_t t = in_stretches(total, few);
    if (t >= total) return;
    const LongShare share = long_share(at, t);
    const LongTensor& x = tab.t[share.tensor];
    auto run = [&](auto n2) __attribute__((always_inline)) {
        constexpr int LOGN2 = decltype(n2)::value, LOGSUB = TOP - LOGN2;
        using G = HalfTile<LOGN2>;
        const uint32_t sub = LOGSUB ? (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / G::NT) : 0u, pp0 = ((share.blk << LOGSUB) + sub) * G::PAIRS;
        fwd_b_pairs<LOGN2, false, TOP>(mid + long_mid(x), x.logM, spec + long_spec(x, share.tensor), tb, hist + (size_t)share.tensor * kHistBins, pp0,
                                       share.blk == 0, reinterpret_cast<uint32_t*>(smem), threadIdx.x, 1.0f);
    };
    const int rows = x.logM / 2;
    if (rows == 7) return run(std::integral_constant<int, 7>{});
    if (rows == 8) return run(std::integral_constant<int, 8>{});
    if (TOP == 9 || rows == 9) return run(std::integral_constant<int, 9>{});
    if constexpr (TOP == 10) run(std::integral_constant<int, 10>{});
}

// Inverse pass B: undo the split, inverse N2-point FFTs over k2, times conj W_M^(n2 k1).
// PAIR: the spectrum is read in the paired order (the codec's own buffer), otherwise in natural bin order.
// HALF (PAIR only): spectrum and intermediate are binary16 pairs.
template <int LOGN2, int LOGE, bool PAIR, bool HALF>
__device__ __forceinline__ void inv_b_workgroup(uint32_t blk, uint32_t nblk, const typename Cx<HALF>::One* __restrict__ spec,
                                                uint32_t sstride, int logM, typename Cx<HALF>::One* __restrict__ mid,
                                                const Tables& tb, uint32_t total, uint32_t per_wg, float mid_scale)
{
    static_assert(PAIR || !HALF, "binary16 storage is the codec's own");
    using One = typename Cx<HALF>::One;
    using Two = typename Cx<HALF>::Two;
    constexpr int NT = tile_lanes(LOGE), PER2 = kLanePairs;
    constexpr int N2 = 1 << LOGN2, LOGT = LOGE - LOGN2, ELEMS = 1 << LOGE;
    constexpr int LOGP = LOGT - 1, P = 1 << LOGP;
    static_assert(LOGT >= 1 && NT % P == 0, "a lane keeps one slot pair");
    extern __shared__ float2 smem[];
    float2* d = smem;
    float2* tw = smem + ELEMS;
    const int tid0 = threadIdx.x;
    const int logN1 = logM - LOGN2;
    const uint32_t M = 1u << logM, N1 = 1u << logN1, tiles = N1 >> LOGT;
    // runs differ by at most one tile: the first total - per_wg * nblk workgroups take one more
    const uint32_t extra = total - per_wg * nblk;
    uint32_t t = blk * per_wg + (blk < extra ? blk : extra);
    const uint32_t tend = t + per_wg + (blk < extra ? 1u : 0u);
    if (t >= tend) return;
    load_stage_twiddles<LOGN2, NT>(tw, tb, tid0);
    constexpr int DK = NT >> LOGP;
    static_assert(PER2 <= 8, "twiddle recurrence is anchored once");

    Two r[PER2];
    One xnyq;                // Nyquist bin of the chunk of the tile held in r
    float2 base_a, base_b;   // split twiddles of that tile
    constexpr int PARTS = portions<LOGN2 - 3, kSpreadIB>();
    // part < 0: the whole tile; otherwise the loads q with q * PARTS / PER2 == part (the look-ups go with part 0)
    auto load_tile = [&](uint32_t tile, int tid, bool live, int part = -1) {
        const int p = tid & (P - 1), kq0 = tid >> LOGP;
        const One* X = spec + (live ? (size_t)(tile / tiles) * (size_t)sstride : 0);
        const uint32_t pp = tile_in_chunk(tile, tiles) * P + p;
        const uint32_t ka = pp, kb = mirror_row(pp, N1);
        if (part <= 0) {
            base_a = twiddle(tb, (ka + ((uint32_t)kq0 << logN1)) << (21 - logM));
            base_b = twiddle(tb, (kb + ((uint32_t)kq0 << logN1)) << (21 - logM));
        }
        if constexpr (PAIR) {
            const Two* X4 = reinterpret_cast<const Two*>(X);
#pragma unroll
            for (int q = 0; q < PER2; ++q)
                if (part < 0 || q * PARTS / PER2 == part) r[q] = X4[live ? ((uint32_t)(kq0 + q * DK) << (logN1 - 1)) + pp : 0u];
        } else {
#pragma unroll
            for (int q = 0; q < PER2; ++q) {
                if (!(part < 0 || q * PARTS / PER2 == part)) continue;
                const uint32_t o = (uint32_t)(kq0 + q * DK) << logN1;
                r[q] = join(X[live ? ka + o : 0u], X[live ? kb + o : 0u]);
            }
        }
        if (part <= 0) xnyq = X[live ? M : 0u];
    };
    auto fill = [&](int tid) {
        const int p = tid & (P - 1), kq0 = tid >> LOGP;
#pragma unroll
        for (int q = 0; q < PER2; ++q) lds_store2<LOGT>(d, kq0 + q * DK, 2 * p, cx_load(r[q]));
    };
    load_tile(t, tid0, true);
    fill(tid0);
    __syncthreads();
    for (;;) {
        const int tid = opaque_lane(tid0);
        const int p = tid & (P - 1), kq0 = tid >> LOGP;
        const uint32_t pp = tile_in_chunk(t, tiles) * P + p;
        const uint32_t ka = pp, kb = mirror_row(pp, N1);
        const bool self = pp == 0;
        // partners of all pairs first (one batch of LDS reads), then the arithmetic: no branches in between
        float2 pa[PER2], pb[PER2];
#pragma unroll
        for (int q = 0; q < PER2; ++q) {
            const int k2 = kq0 + q * DK, k2p = N2 - 1 - k2;
            const int ia = self ? sw_idx<LOGT>((N2 - k2) & (N2 - 1), 2 * p) : sw_idx<LOGT>(k2p, 2 * p + 1);
            const int ib = self ? sw_idx<LOGT>(k2p, 2 * p + 1) : sw_idx<LOGT>(k2p, 2 * p);
            pa[q] = d[ia];
            pb[q] = d[ib];
        }
        float4 z[PER2];
#pragma unroll
        for (int q = 0; q < PER2; ++q) {
            const float2 wq = make_float2(kW32re[2 * q * kSplitStep], kW32im[2 * q * kSplitStep]);
            const float4 rq = cx_load(r[q]);
            float2 a0 = lo2(rq), b0 = pa[q];
            if (q == 0) {  // k2 = 0 only here; imaginary parts of the DC and Nyquist bins are ignored
                const bool dc = self && kq0 == 0;
                b0 = dc ? make_float2(cx_load(xnyq).x, 0.f) : b0;
                a0.y = dc ? 0.f : a0.y;
            }
            z[q] = join(split_inv(a0, b0, cmul(base_a, wq)), split_inv(hi2(rq), pb[q], cmul(base_b, wq)));
        }
        __syncthreads();
        // z[q] are rows kq0 + q * N2/8 of this lane's slot pair: the first inverse radix-8 stage runs here
        static_assert(PER2 == 8 && DK == N2 / 8, "a lane's values are the inputs of two radix-8 butterflies");
        first_stage_store<LOGT, true>(d, kq0, 2 * p, z);
        __syncthreads();
        // store-loop twiddles of this tile, then split twiddles and data of the next one
        const int sh = 22 - logM;
        const float2 ratio_a = twiddle(tb, ((uint32_t)DK * ka) << sh);
        const float2 ratio_b = twiddle(tb, ((uint32_t)DK * kb) << sh);
        float2 cur_a = twiddle(tb, ((uint32_t)kq0 * ka) << sh);
        float2 cur_b = twiddle(tb, ((uint32_t)kq0 * kb) << sh);
        if constexpr (HALF) {  // keeps the unnormalised partial sums inside binary16's range (exact power of two)
            cur_a = make_float2(cur_a.x * mid_scale, cur_a.y * mid_scale);
            cur_b = make_float2(cur_b.x * mid_scale, cur_b.y * mid_scale);
        }
        const bool more = t + 1 < tend;
        load_tile(more ? t + 1 : t, tid, more, 0);
        run_fft_between<LOGN2, LOGT, NT, true, 3>(d, tw, tid, [&](int k) {
            if (k + 1 < PARTS) load_tile(more ? t + 1 : t, tid, more, k + 1);
        });
        Two* dst = reinterpret_cast<Two*>(mid + (size_t)(t / tiles) * (size_t)M);
#pragma unroll
        for (int q = 0; q < PER2; ++q) {
            const uint32_t n2 = (uint32_t)(kq0 + q * DK);
            const float4 v = lds_load2<LOGT>(d, (int)n2, 2 * p);
            dst[n2 * (N1 >> 1) + pp] = cx_store<HALF>(join(cmulc(lo2(v), cur_a), cmulc(hi2(v), cur_b)));
            cur_a = cmul(cur_a, ratio_a);
            cur_b = cmul(cur_b, ratio_b);
        }
        if (!more) break;
        ++t;
        __syncthreads();
        fill(tid);
        __syncthreads();
    }
}

template <int LOGN2, int LOGE, bool PAIR, bool HALF>
__global__ __launch_bounds__(tile_lanes(LOGE)) void k_inv_b(const typename Cx<HALF>::One* __restrict__ spec, uint32_t sstride, int logM,
                                               typename Cx<HALF>::One* __restrict__ mid, Tables tb, uint32_t total,
                                               uint32_t per_wg, float mid_scale, const uint32_t* __restrict__ only_if)
{
    if (only_if && *only_if == 0u) return;  // stand-by launch behind a fused kernel that did finish
    inv_b_workgroup<LOGN2, LOGE, PAIR, HALF>(blockIdx.x, gridDim.x, spec, sstride, logM, mid, tb, total, per_wg, mid_scale);
}

// Inverse pass A: inverse N1-point FFTs over k1 for a tile of columns n2; writes the real samples to out[first .. first + n),
// chunk by chunk.  `aligned`: `out` is 16-byte aligned.
// ONCE: what it reads and writes passes the caches by.
template <int LOGN1, int LOGE, bool HALF, bool ONCE>
__device__ __forceinline__ void inv_a_workgroup(uint32_t blk, const typename Cx<HALF>::One* __restrict__ mid, int logM,
                                                float* __restrict__ out, size_t n, const Tables& tb, bool aligned,
                                                uint32_t total, uint32_t per_wg, int glog, float gain)
{
    using Two = typename Cx<HALF>::Two;
    constexpr int NT = tile_lanes(LOGE), PER2 = kLanePairs;
    constexpr int N1 = 1 << LOGN1, LOGT = LOGE - LOGN1, TA = 1 << LOGT, ELEMS = 1 << LOGE;
    constexpr int HP = N1 / 2, LOGHP = LOGN1 - 1;
    static_assert(LOGT >= 2 && (NT % (TA / 2)) == 0, "tile shape");
    extern __shared__ float2 smem[];
    float2* d = smem;
    float2* tw = smem + ELEMS;
    const int tid0 = threadIdx.x;
    const uint32_t M = 1u << logM, N2 = M >> LOGN1, tiles = N2 >> LOGT;
    uint32_t t, tend;
    if (!grouped_run(blk, total, per_wg, glog, t, tend)) return;
    const uint32_t tstep = 1u << glog;
    load_stage_twiddles<LOGN1, NT>(tw, tb, tid0);

    Two r[PER2];
    constexpr int PARTS = portions<LOGN1, kSpreadIA>();
    // part < 0: the whole tile; otherwise the loads q with q * PARTS / PER2 == part
    auto load_tile = [&](uint32_t tile, int tid, bool live, int part = -1) {
        const Two* src = reinterpret_cast<const Two*>(mid + (live ? (size_t)(tile / tiles) * (size_t)M : 0));
        const uint32_t col0 = tile_in_chunk(tile, tiles) << LOGT;
#pragma unroll
        for (int q = 0; q < PER2; ++q) {
            if (!(part < 0 || q * PARTS / PER2 == part)) continue;
            const int w = tid + q * NT, kp = w & (HP - 1), col = w >> LOGHP;
            r[q] = load_maybe_once<ONCE>(src + (live ? (uint32_t)(col0 + col) * HP + kp : 0u));
        }
    };
    auto fill = [&](int tid) {
#pragma unroll
        for (int q = 0; q < PER2; ++q) {
            const int w = tid + q * NT, kp = w & (HP - 1), col = w >> LOGHP;
            const float4 rq = cx_load(r[q]);
            d[sw_idx<LOGT>(kp, col)] = lo2(rq);
            d[sw_idx<LOGT>((int)mirror_row((uint32_t)kp, N1), col)] = hi2(rq);
        }
    };
    load_tile(t, tid0, true);
    fill(tid0);
    __syncthreads();
    const float scale = gain * (1.0f / (float)(2u * M));
    for (;;) {
        const int tid = opaque_lane(tid0);
        const bool more = t + tstep < tend;
        load_tile(more ? t + tstep : t, tid, more, 0);
        run_fft_between<LOGN1, LOGT, NT, true, 0>(d, tw, tid, [&](int k) {
            if (k + 1 < PARTS) load_tile(more ? t + tstep : t, tid, more, k + 1);
        });
        const Span sp = chunk_span(0, n, t / tiles, 2 * (size_t)M);
        const size_t cbase = sp.first;
        const uint32_t col0 = tile_in_chunk(t, tiles) << LOGT;
        if (aligned && (cbase & 3u) == 0 && (cbase + 2 * (size_t)M <= sp.limit || (sp.limit & 3u) == 0)) {
            // 16-byte pieces, each inside the output or outside it
            float4* dst = reinterpret_cast<float4*>(out + cbase);
            const size_t left = sp.limit > cbase ? (sp.limit - cbase) >> 2 : 0;
            const uint32_t quads = left < (size_t)(M >> 1) ? (uint32_t)left : M >> 1;
#pragma unroll
            for (int q = 0; q < PER2; ++q) {
                const int w = tid + q * NT, bp = w & (TA / 2 - 1), n1 = w >> (LOGT - 1);
                const uint32_t i = (uint32_t)n1 * (N2 >> 1) + (col0 >> 1) + bp;
                const float4 v = lds_load2<LOGT>(d, n1, 2 * bp);
                if (i < quads) store_maybe_once<ONCE>(dst + i, make_float4(v.x * scale, v.y * scale, v.z * scale, v.w * scale));
            }
        } else {
#pragma unroll
            for (int q = 0; q < PER2; ++q) {
                const int w = tid + q * NT, bp = w & (TA / 2 - 1), n1 = w >> (LOGT - 1);
                const float4 v = lds_load2<LOGT>(d, n1, 2 * bp);
                const size_t gi = cbase + 2 * ((size_t)n1 * N2 + col0 + 2 * bp);
                store_pair(out, gi, sp.limit, make_float2(v.x * scale, v.y * scale));
                store_pair(out, gi + 2, sp.limit, make_float2(v.z * scale, v.w * scale));
            }
        }
        if (!more) break;
        t += tstep;
        __syncthreads();
        fill(tid);
        __syncthreads();
    }
}

template <int LOGN1, int LOGE, bool HALF, bool ONCE>
__global__ __launch_bounds__(tile_lanes(LOGE)) void k_inv_a(const typename Cx<HALF>::One* __restrict__ mid, int logM,
                                               float* __restrict__ out, size_t n, Tables tb, bool aligned, uint32_t total,
                                               uint32_t per_wg, int glog, float gain, const uint32_t* __restrict__ only_if)
{
    if (only_if && *only_if == 0u) return;  // stand-by launch behind a fused kernel that did finish
    inv_a_workgroup<LOGN1, LOGE, HALF, ONCE>(blockIdx.x, mid, logM, out, n, tb, aligned, total, per_wg, glog, gain);
}

// Inverse pass A with a tile in half of the LDS, as fwd_a_split: the same radices, twiddles and order of operations as inv_a_workgroup.  The last
// stage's butterflies are dealt out so that a lane has both of two adjacent columns and stores 16 bytes from its registers.
// Four tiles of 2^13 points to a compute unit where the persistent kernel has two, and no rounds of runs of equal length that end together.
// Receivers in us, persistent / this, by number of tiles of 2^14; behind a semicolon with a kernel after each call that reads the output:
//   columns of 2^9, through the caches: 2^19 8.4 M samples 43.5 / 39.5, 25.6 M 81.5 / 75.1; 2^18 20 M 63.0 / 59.1; past them: 2^19 1024 97.5 / 90.8; 171.4 / 166.4, 1920
//     192.1 / 174.7; 330.4 / 296.7, binary16 1920 156.5 / 134.6; 291.0 / 268.1, 2^18 1600 157.3 / 148.6;
//   columns of 2^10, through the caches, persistent / this with tiles of 2^14 / of 2^13: 256 43.7 / 40.6 / 40.1, 512 60.6 / 59.0 / 57.0, 640 80.5 / 81.0 / 74.6, 768
//     79.2 / 79.5 / 78.1; past them, persistent / this with 2^14: 2^20 1024 95.1 / 93.1; 173.2 / 171.1, 1280 114.8 / 113.0; 206.7 / 203.4, 1536 134.4 / 135.3; 256.4 / 240.4,
//     1920 191.9 / 184.9; 329.9 / 304.7, 3840 380.7 / 357.8; 637.0 / 608.7; 2^21 1024 103.6 / 105.2; 178.7 / 179.6, 1280 127.7 / 126.7; 223.8 / 216.7, 1920 207.9 /
//     201.1; 346.8 / 327.9; binary16 2^20 1024 89.7 / 85.5; 164.0 / 159.2, 1920 151.9 / 147.0; 281.5 / 276.3;
//   columns of 2^11, through the caches: 256 51.1 / 48.6, 384 64.2 / 60.7, 512 70.5 / 69.1, 640 91.1 / 90.9; 127.6 / 129.5, 768 97.8 / 98.5; 147.7 / 149.8, 896 114.2 / 114.1;
//     187.2 / 184.9, 1024 120.5 / 127.2; 208.5 / 211.3; past them: 1024 117.8 / 118.6; 194.7 / 194.1, 1152 135.8 / 131.7; 222.6 / 213.8, 1920 231.3 / 221.2; 371.7 / 352.0,
//     4224 537.7 / 492.0; 832.3 / 785.9; binary16 through the caches 640 85.8 / 81.6; 131.6 / 127.0, 768 91.2 / 88.3; 132.4 / 130.5, 896 108.6 / 102.7; 162.0 / 158.2, past
//     them 1024 113.8 / 114.3; 189.5 / 191.9, 1280 136.2 / 134.6; 229.3 / 224.3, 4224 428.8 / 394.0; 733.9 / 689.9;
//   columns of 2^8, two stages: 10 M 44.0 / 44.0, 45 M 134 / 150.
constexpr size_t kSplitInverse10 = 1024;  // fewer tiles: of 2^13; else of 2^14
constexpr size_t kSplitInverse11 = 640;   // binary32 through the caches: from here on the persistent kernel
template <int LOGN1, int LOGE>
struct SplitInverse {
    static constexpr int N1 = 1 << LOGN1, LOGT = LOGE - LOGN1, T = 1 << LOGT, NT = tile_lanes(LOGE), HP = N1 / 2, LOGHP = LOGN1 - 1;
    static constexpr size_t kLds = ((size_t)sizeof(float) << LOGE) + N1 * sizeof(float2);
    static constexpr int RL1 = stage_radix_log(LOGN1), RL2 = stage_radix_log(LOGN1 - RL1), RL3 = LOGN1 - RL1 - RL2;
    static_assert(T >= 8 && T <= 32 && RL1 >= 3 && (RL3 == 3 || (RL3 == 0 && RL2 == 4)), "three stages, the last of radix 8, or two (columns of 2^8, in tensors' launches)");
    // Rows and columns as loaded: 64 lanes have one column of 64 neighbouring rows, and then all columns of 64 / T of them
    static __device__ __forceinline__ int loaded(int i, int b) { return (i << LOGT) + (b ^ ((i >> (6 - LOGT)) & (T - 1))); }
    // between the first two stages: rows a radix apart, then neighbouring ones
    static __device__ __forceinline__ int staged(int i, int b) { return ((i ^ ((i >> RL1) & (64 / T - 1))) << LOGT) + b; }
    static __device__ __forceinline__ int butterfly_of(int tid, int q) { return (tid >> LOGT) + q * (NT >> LOGT); }
    // row(q) = the butterfly's number; points q * RHO + t
    template <int NS_LOG, int RL, typename Row>
    static __device__ __forceinline__ void stage(float2 (&v)[16], const float2* tw, Row&& row)
    {
        constexpr int RHO = 1 << RL;
#pragma unroll
        for (int q = 0; q < 16 / RHO; ++q) {
            if constexpr (NS_LOG > 0) {
                const int k = row(q) & ((1 << NS_LOG) - 1);
#pragma unroll
                for (int t = 1; t < RHO; ++t) v[q * RHO + t] = cmulc(v[q * RHO + t], tw[(t * k) << (LOGN1 - NS_LOG - RL)]);
            }
            butterfly<RL, true>(v + q * RHO);
        }
    }
};
// Four neighbouring samples wherever they start, those that are there, in one instruction (receivers: 37 tensors of up to 4 M samples 101.5 -> 90.9 us, 33 of up to 1.7 M 71.3 -> 67.3,
// 66 of up to 2.4 M 105.7 -> 101.4).
__device__ __forceinline__ void store_floats(float* __restrict__ out, size_t gi, size_t limit, float4 z)
{
    if (gi + 4 <= limit) {
        *reinterpret_cast<Floats4*>(out + gi) = Floats4{z.x, z.y, z.z, z.w};
    } else {
        if (gi < limit) out[gi] = z.x;
        if (gi + 1 < limit) out[gi + 1] = z.y;
        if (gi + 2 < limit) out[gi + 2] = z.z;
    }
}
// TOP: 2^(TOP - LOGE) tiles beside each other, each with words d of its own, share the stage twiddles
template <int LOGN1, int LOGE, bool HALF, bool ONCE, int TOP = LOGE>
__device__ __forceinline__ void inv_a_split(const typename Cx<HALF>::One* __restrict__ mid, int logM, float* __restrict__ out, const Span& sp, bool quads,
                                            const Tables& tb, uint32_t col0, float* d, float2* tw, int lane, float gain)
{
    using G = SplitInverse<LOGN1, LOGE>;
    using Two = typename Cx<HALF>::Two;
    constexpr int N1 = G::N1, HP = G::HP, T = G::T, LOGT = G::LOGT, NT = G::NT, RHO1 = 1 << G::RL1, RHO2 = 1 << G::RL2;
    const uint32_t M = 1u << logM, N2 = M >> LOGN1;
    const int tid = lane & (NT - 1), b = tid & (T - 1), bp = tid & (T / 2 - 1), j2 = tid >> (LOGT - 1);
    float2 v[16];
    {
        Two raw[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int w = tid + q * NT, kp = w & (HP - 1), col = w >> G::LOGHP;
            raw[q] = load_maybe_once<ONCE>(reinterpret_cast<const Two*>(mid) + ((col0 + (uint32_t)col) * (uint32_t)HP + (uint32_t)kp));
        }
        load_stage_twiddles<LOGN1, tile_lanes(TOP)>(tw, tb, lane);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float4 z = cx_load(raw[q]);
            v[2 * q] = lo2(z);
            v[2 * q + 1] = hi2(z);
        }
    }
    float x[16];
    // component by component: to(n) <- v[n], then v[n] <- from(n)
    // (addresses are computed again for the second component: kept, they spill)
    auto exchange = [&](auto to, auto get) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < 16; ++n) d[to(n, tid)] = v[n].x;
        __syncthreads();
        get(x, tid);
        __syncthreads();
        const int again = opaque_lane(tid);
#pragma unroll
        for (int n = 0; n < 16; ++n) d[to(n, again)] = v[n].y;
        __syncthreads();
        float y[16];
        get(y, again);
#pragma unroll
        for (int n = 0; n < 16; ++n) v[n] = make_float2(x[n], y[n]);
    };
    exchange(
        [&](int n, int tid) __attribute__((always_inline)) {
            const int w = tid + (n >> 1) * NT, kp = w & (HP - 1);
            return G::loaded(n & 1 ? (int)mirror_row((uint32_t)kp, N1) : kp, w >> G::LOGHP);
        },
        [&](float (&to)[16], int tid) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < 16; ++n) to[n] = d[G::loaded(G::butterfly_of(tid, n >> G::RL1) + (n & (RHO1 - 1)) * (N1 / RHO1), tid & (T - 1))];
        });
    G::template stage<0, G::RL1>(v, tw, [](int) { return 0; });
    __syncthreads();
    exchange([&](int n, int tid) __attribute__((always_inline)) { return G::staged(G::butterfly_of(tid, n >> G::RL1) * RHO1 + (n & (RHO1 - 1)), tid & (T - 1)); },
             [&](float (&to)[16], int tid) __attribute__((always_inline)) {
#pragma unroll
                 for (int n = 0; n < 16; ++n) to[n] = d[G::staged(G::butterfly_of(tid, n >> G::RL2) + (n & (RHO2 - 1)) * (N1 / RHO2), tid & (T - 1))];
             });
    G::template stage<G::RL1, G::RL2>(v, tw, [&](int q) __attribute__((always_inline)) { return G::butterfly_of(tid, q); });
    const float scale = gain * (1.0f / (float)(2u * M));
    const size_t left = sp.limit > sp.first ? (sp.limit - sp.first) >> 2 : 0;
    const uint32_t end = left < (size_t)(M >> 1) ? (uint32_t)left : M >> 1;  // 16-byte pieces that exist
    if constexpr (G::RL3 == 0) {
        float2* dst = reinterpret_cast<float2*>(out + sp.first);
#pragma unroll
        for (int n = 0; n < 16; ++n) {
            const uint32_t i = (uint32_t)((tid >> LOGT) + n * (N1 / 16)) * N2 + col0 + (uint32_t)b;
            const float2 z = make_float2(v[n].x * scale, v[n].y * scale);
            if (!quads)
                store_pair(out, sp.first + 2 * (size_t)i, sp.limit, z);
            else if (i < 2 * end)
                dst[i] = z;
        }
        return;
    }
    __syncthreads();
    exchange(
        [&](int n, int tid) __attribute__((always_inline)) {
            const int j = G::butterfly_of(tid, n >> G::RL2);
            return ((((j >> G::RL1) << (G::RL1 + G::RL2)) + (j & (RHO1 - 1)) + ((n & (RHO2 - 1)) << G::RL1)) << LOGT) + (tid & (T - 1));
        },
        [&](float (&to)[16], int tid) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float2 two = *reinterpret_cast<const float2*>(d + (((tid >> (LOGT - 1)) + t * (N1 / 8)) << LOGT) + 2 * (tid & (T / 2 - 1)));
                to[t] = two.x;
                to[8 + t] = two.y;
            }
        });
    G::template stage<LOGN1 - 3, 3>(v, tw, [&](int) __attribute__((always_inline)) { return j2; });
    if (quads) {
        float4* dst = reinterpret_cast<float4*>(out + sp.first);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint32_t i = (uint32_t)(j2 + t * (N1 / 8)) * (N2 >> 1) + (col0 >> 1) + (uint32_t)bp;
            if (i < end) store_maybe_once<ONCE>(dst + i, make_float4(v[t].x * scale, v[t].y * scale, v[8 + t].x * scale, v[8 + t].y * scale));
        }
    } else {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const size_t gi = sp.first + 2 * ((size_t)(j2 + t * (N1 / 8)) * N2 + col0 + 2 * bp);
            store_floats(out, gi, sp.limit, make_float4(v[t].x * scale, v[t].y * scale, v[8 + t].x * scale, v[8 + t].y * scale));
        }
    }
}
template <int LOGN1, int LOGE, bool HALF, bool ONCE>
__global__ __launch_bounds__(tile_lanes(LOGE)) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_inv_a_split(
    const typename Cx<HALF>::One* __restrict__ mid, int logM, float* __restrict__ out, size_t n, Tables tb, bool aligned, uint32_t total, float gain,
    const uint32_t* __restrict__ only_if)
{
    using G = SplitInverse<LOGN1, LOGE>;
    if (only_if && *only_if == 0u) return;  // stand-by launch behind a fused kernel that did finish
    extern __shared__ float2 smem[];
    const uint32_t t = in_stretches(total);
    if (t >= total) return;
    const int log_tiles = logM - LOGE;
    const uint32_t c = t >> log_tiles;
    const Span sp = chunk_span(0, n, c, (size_t)2 << logM);
    const bool quads = aligned && (sp.first + ((size_t)2 << logM) <= n || (n & 3u) == 0);
    inv_a_split<LOGN1, LOGE, HALF, ONCE>(mid + ((size_t)c << logM), logM, out, sp, quads, tb, (t & ((1u << log_tiles) - 1u)) << G::LOGT,
                                   reinterpret_cast<float*>(smem), smem + (1 << LOGE) / 2, threadIdx.x, gain);
}

// ------------------------------------------------- tensors of different lengths ----
// The four passes over the tensors of one LongTable: a workgroup finds the tensor it belongs to and does what a workgroup of
// the uniform kernels does for a call with that tensor as its only chunk.  Rows and columns of any length share a launch
// (the longest of either decides the LDS), so a call with tensors of seven lengths is four launches instead of 28, and short
// tensors fill the compute units that the long ones leave.
// Measured, ResNet-50's 161 tensors (49 of them long, of seven lengths), sender and receiver: seven launch sets on four
// streams 579 us, one 451; the three long tensors of ResNet-20, all of 2^16, stay as they were.
constexpr int log_rows(int logM) { return logM / 2; }           // log2 N2
constexpr int kLongMax = kMaxLogL - 1;                            // log2 M

constexpr int kTallTile = 14;  // of rows of 2^10, where a launch has no others

// A workgroup has 2^TOP points of a tensor: one tile, or with TOP = 14 two of columns of up to 2^10 (fewer tensors: k_fwd_a_long).  Bound by memory, and by what few tiles to a
// compute unit leave idle: a tile in half of the LDS has twice as many in flight as a persistent workgroup with one in all of it, which most launch
// sets of tensors, with one or two tiles to a workgroup, paid for without having a next tile to load ahead; and tensors that start anywhere
// are read 16 bytes at a time.  Pass in us, the persistent kernel / this: ResNet-50's 161 tensors 77 / 74, 100 of 10 to 2.4 M samples 58.6 / 53.4, 200
// 138.5 / 110; senders 240 / 234, 193 / 181, 412 / 380, 24 tensors of 4.2 M padded samples 117 / 109.  Tiles of 2^14 for columns of 2^10: equal.
template <int TOP>
__global__ __launch_bounds__(tile_lanes(TOP)) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_fwd_a_split_long(
    const float* __restrict__ in, float2* __restrict__ mid, Tables tb, uint32_t total, uint32_t step, uint32_t* __restrict__ zero_ptr, uint32_t zero_words,
    LongTable tab, LongStarts at)
{
    extern __shared__ float2 smem[];
    for (uint32_t i = blockIdx.x * tile_lanes(TOP) + threadIdx.x; i < zero_words; i += gridDim.x * tile_lanes(TOP)) zero_ptr[i] = 0u;
    const uint32_t t = in_turned_stretches(total, step);
    if (t >= total) return;
    const LongShare share = long_share(at, t);
    fwd_a_split_tensor<TOP>(tab.t[share.tensor], share.blk, in, mid, tb);
}

// rows of 2^10 in tiles of 2^14, or few tensors of any rows in tiles of 2^13
template <int LOGE>
__global__ __launch_bounds__(tile_lanes(LOGE)) void k_fwd_b_long(const float2* __restrict__ mid, float2* __restrict__ spec, Tables tb,
                                                                uint32_t* __restrict__ hist, uint32_t per_wg, LongTable tab, LongStarts at)
{
    const LongShare share = long_share(at);
    const LongTensor& x = tab.t[share.tensor];
    auto run = [&](auto n2) __attribute__((always_inline)) {
        const uint32_t total = power_tiles(x.logM, LOGE), per = per_wg < total ? per_wg : total;
        fwd_b_workgroup<decltype(n2)::value, LOGE, true, false>(share.blk, total / per, mid + long_mid(x), x.logM, spec + long_spec(x, share.tensor), 0u,
                                                                tb, hist + (size_t)share.tensor * kHistBins, total, per, 1.0f);
    };
    if constexpr (LOGE < kTallTile) {
        const int rows = log_rows(x.logM);
        if (rows == 7) return run(std::integral_constant<int, 7>{});
        if (rows == 8) return run(std::integral_constant<int, 8>{});
        if (rows == 9) return run(std::integral_constant<int, 9>{});
    }
    run(std::integral_constant<int, 10>{});
}

template <int LOGE>
__global__ __launch_bounds__(tile_lanes(LOGE)) void k_inv_b_long(const float2* __restrict__ spec, float2* __restrict__ mid, Tables tb,
                                                uint32_t per_wg, LongTable tab, LongStarts at)
{
    const LongShare share = long_share(at);
    const LongTensor& x = tab.t[share.tensor];
    const int logM = x.logM;
    auto run = [&](auto n2) __attribute__((always_inline)) {
        const uint32_t total = power_tiles(logM, LOGE), per = per_wg < total ? per_wg : total;
        inv_b_workgroup<decltype(n2)::value, LOGE, true, false>(share.blk, total / per, spec + long_spec(x, share.tensor), 0u, logM,
                                                                mid + long_mid(x), tb, total, per, 1.0f);
    };
    const int rows = log_rows(logM);
    if constexpr (LOGE == 13) {
        if (rows == 7) return run(std::integral_constant<int, 7>{});
        if (rows == 8) return run(std::integral_constant<int, 8>{});
        if (rows == 9) return run(std::integral_constant<int, 9>{});
    }
    run(std::integral_constant<int, 10>{});
}

// A workgroup has 2^TOP points of a tensor: one tile, or with TOP = 14 two of columns of less than 2^10.  Eight waves a SIMD, eleven or twelve registers spilled with
// three or four transforms in one kernel; none with six (TOP 13) or four waves: receivers of 100 tensors 138.5 / 158.5, 150 164.7 / 191.3, 60 of 2^20 208.7 / 226.1, five of
// 3 M 84.8 / 96.2.
template <int TOP>
__global__ __launch_bounds__(tile_lanes(TOP)) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_inv_a_split_long(
    const float2* __restrict__ mid, float* __restrict__ out, Tables tb, bool aligned, uint32_t total, LongTable tab, LongStarts at)
{
    extern __shared__ float2 smem[];
    const uint32_t t = in_stretches(total);
    if (t >= total) return;
    const LongShare share = long_share(at, t);
    const LongTensor& x = tab.t[share.tensor];
    const int logM = x.logM;
    const Span sp = chunk_span((size_t)x.goff, x.glen, 0, 0);
    const bool quads = aligned && (x.goff & 3u) == 0 && (x.glen & 3u) == 0;
    auto run = [&](auto n1) __attribute__((always_inline)) {
        constexpr int LOGN1 = decltype(n1)::value, LOGE = LOGN1 >= 10 ? TOP : 13;
        using G = SplitInverse<LOGN1, LOGE>;
        const uint32_t sub = LOGE < TOP ? (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / G::NT) : 0u, tile = (share.blk << (TOP - LOGE)) + sub;
        inv_a_split<LOGN1, LOGE, false, false, TOP>(mid + long_mid(x), logM, out, sp, quads, tb, tile << G::LOGT, reinterpret_cast<float*>(smem) + (sub << LOGE),
                                            smem + (1 << TOP) / 2, (int)threadIdx.x, 1.0f);
    };
    const int columns = log_columns(logM);
    if (columns == 8) return run(std::integral_constant<int, 8>{});
    if (columns == 9) return run(std::integral_constant<int, 9>{});
    if (TOP == 13 || columns == 10) return run(std::integral_constant<int, 10>{});
    if constexpr (TOP == 14) run(std::integral_constant<int, 11>{});
}

// ---------------------------------------------------------------- launch ----
template <typename K>
hipError_t set_lds(K kernel, size_t bytes)
{
    if (bytes <= 48 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
}

// persistent grid: workgroups walk contiguous runs of tiles; two of them are resident per compute unit (512 on
// the chip), and a kernel may ask for a few rounds of that when shorter runs balance better
struct Grid {
    uint32_t wgs, per_wg;
};
// Every workgroup takes per_wg tiles and the first total - per_wg * wgs of them one more.  With 512 workgroups
// (256 compute units x 2 resident) the two workgroups of a compute unit are b and b + 256, so the longer runs pair
// up with the shorter ones and every compute unit gets the same number of tiles.
Grid persistent_grid(size_t total, uint32_t kMaxWgs = 512)
{
    Grid g;
    g.wgs = (uint32_t)(total < kMaxWgs ? total : kMaxWgs);
    g.per_wg = (uint32_t)(total / g.wgs);
    return g;
}

// pass A: 2^glog workgroups (b, b+8, ...) share a run of aligned tile groups; per_wg counts tile groups and wgs
// is a multiple of 8 * 2^glog
// most workgroups of a launch: the figures below are for two resident workgroups per compute unit
constexpr uint32_t most_wgs(int loge, uint32_t with_two) { return loge == 13 ? with_two : with_two / 2; }
constexpr uint32_t kPassAWgs = 2048;  // most workgroups the forward pass A is cut into
Grid grouped_grid(size_t groups, int glog, uint32_t kMaxWgs = 512)
{
    Grid g;
    const uint32_t wg_groups = kMaxWgs >> glog;
    g.per_wg = (uint32_t)((groups + wg_groups - 1) / wg_groups);
    const uint32_t used = (uint32_t)((groups + g.per_wg - 1) / g.per_wg);
    const uint32_t unit = 8u << glog;
    g.wgs = (((used << glog) + unit - 1) / unit) * unit;
    return g;
}

template <int LOGN1, int LOGE, bool HALF>
hipError_t fwd_a_halved(const float* in, size_t n, int logM, size_t C, typename Cx<HALF>::One* mid, Tables t, uint32_t* zero_ptr,
                        uint32_t zero_words, float in_scale, hipStream_t s)
{
    using G = SplitTile<LOGN1, LOGE>;
    const auto kern = k_fwd_a_split<LOGN1, LOGE, HALF>;
    const hipError_t e = set_lds(kern, G::kLds);
    if (e != hipSuccess) return e;
    const size_t total = C << (logM - LOGE);
    FFTSP_LAUNCH("rfft_pass_a", kern, dim3((unsigned)(8 * ((total + 7) / 8))), dim3(G::NT), G::kLds, s, in, n, logM, mid, t, (uint32_t)total, zero_ptr,
                 zero_words, in_scale);
    return hipGetLastError();
}
// HALF launchers take the same buffer pointers; the kernels read them as binary16 pairs
template <int LOGN1, bool HALF>
hipError_t fwd_a(const float* in, size_t n, int logM, size_t C, float2* mid_f32, Tables t, bool aligned,
                 uint32_t* zero_ptr, uint32_t zero_words, float in_scale, hipStream_t s,
                 const uint32_t* only_if = nullptr)
{
    constexpr int LOGE = kTileFA;
    const size_t lds = ((size_t)(1 << LOGE) + (1 << LOGN1)) * sizeof(float2);
    auto kern = k_fwd_a<LOGN1, HALF>;
    auto* mid = reinterpret_cast<typename Cx<HALF>::One*>(mid_f32);
    hipError_t e = set_lds(kern, lds);
    if (e != hipSuccess) return e;
    if constexpr (LOGN1 == 11)
        if (!only_if && wide_tiles(C, logM) >= kSplitForward<HALF>) return fwd_a_halved<LOGN1, 14, HALF>(in, n, logM, C, mid, t, zero_ptr, zero_words, in_scale, s);
    if constexpr (LOGN1 == 10 && HALF)
        if (!only_if && wide_tiles(C, logM) >= 1024) return fwd_a_halved<LOGN1, 13, HALF>(in, n, logM, C, mid, t, zero_ptr, zero_words, in_scale, s);
    const size_t total = C * (((size_t)1 << (logM - LOGN1)) >> (LOGE - LOGN1));
    constexpr int glog = group_log(LOGE, LOGN1);  // a chunk has at least that many tiles
    // measured: 143 us against 149 with 512; a stand-by launch (only_if) takes the small grid, which leaves sooner
    const Grid g = grouped_grid(total >> glog, glog, most_wgs(LOGE, only_if ? 512 : kPassAWgs));
    FFTSP_LAUNCH(only_if ? "rfft_pass_a_standby" : "rfft_pass_a", kern, dim3(g.wgs), dim3(tile_lanes(LOGE)), lds, s, in, n, logM, mid,
                 t, aligned, (uint32_t)(total >> glog), g.per_wg, glog, zero_ptr, zero_words, in_scale, only_if);
    return hipGetLastError();
}

template <int LOGN2, int LOGE, bool CODEC, bool HALF>
hipError_t fwd_b_tiled(const float2* mid_f32, int logM, size_t C, float2* spec_f32, uint32_t sstride, Tables t, uint32_t* hist,
                 float mid_scale, hipStream_t s, const uint32_t* only_if)
{
    const size_t lds = ((size_t)(1 << LOGE) + (1 << LOGN2)) * sizeof(float2) + kHistLdsWords * sizeof(uint32_t);
    auto kern = k_fwd_b<LOGN2, LOGE, CODEC, HALF>;
    auto* mid = reinterpret_cast<const typename Cx<HALF>::One*>(mid_f32);
    auto* spec = reinterpret_cast<typename Cx<HALF>::One*>(spec_f32);
    hipError_t e = set_lds(kern, lds);
    if (e != hipSuccess) return e;
    const size_t total = C * (((size_t)1 << (logM - LOGN2)) >> (LOGE - LOGN2));
    const Grid g = persistent_grid(total, most_wgs(LOGE, 512));
    FFTSP_LAUNCH(only_if ? "rfft_pass_b_standby" : "rfft_pass_b", kern, dim3(g.wgs), dim3(tile_lanes(LOGE)), lds, s, mid, logM, spec,
                 sstride, t, hist, (uint32_t)total, g.per_wg, mid_scale, only_if);
    return hipGetLastError();
}

template <int LOGN2, int LOGE, bool PAIR, bool HALF>
hipError_t inv_b_tiled(const float2* spec_f32, uint32_t sstride, int logM, size_t C, float2* mid_f32, Tables t, float mid_scale,
                 hipStream_t s, const uint32_t* only_if)
{
    const size_t lds = ((size_t)(1 << LOGE) + (1 << LOGN2)) * sizeof(float2);
    auto kern = k_inv_b<LOGN2, LOGE, PAIR, HALF>;
    auto* spec = reinterpret_cast<const typename Cx<HALF>::One*>(spec_f32);
    auto* mid = reinterpret_cast<typename Cx<HALF>::One*>(mid_f32);
    hipError_t e = set_lds(kern, lds);
    if (e != hipSuccess) return e;
    const size_t total = C * (((size_t)1 << (logM - LOGN2)) >> (LOGE - LOGN2));
    const Grid g = persistent_grid(total, most_wgs(LOGE, only_if ? 512 : 1536));  // measured: 117 us against 126 with 512
    FFTSP_LAUNCH(only_if ? "irfft_pass_b_standby" : "irfft_pass_b", kern, dim3(g.wgs), dim3(tile_lanes(LOGE)), lds, s, spec, sstride,
                 logM, mid, t, (uint32_t)total, g.per_wg, mid_scale, only_if);
    return hipGetLastError();
}

// Large outputs pass the caches by, and so do the last reads of the intermediate: the two do not fit the 256 MB cache together, and what
// is kept of them there has to be written back, or made room for, under the kernels that come next, a caller's that reads the output among them.
// Calls in us, all through the caches / this, alone and with a kernel behind each call that reads the output and updates as many weights:
//   2^20 34 M samples receiver 118.6 / 99.5 and 187.9 / 178.1, 45 M 146.4 / 130.2 and 239.8 / 232.1, 62 M 208.8 / 193.6 and 334.4 / 328.8, step 531.6 / 511.5
//   and 658.9 / 640.3, binary16 step 424.4 / 402.6 and 558.4 / 534.6;  2^22 100 M receiver 409.9 / 350.6 and 642.6 / 550.9, 138 M step 1309.9 / 1247.2 and
//   1622.4 / 1529.1;  2^16 40 M receiver 122.9 / 103.5 and 209.1 / 199.8.  A kernel that reads and writes elsewhere: 62 M step 611.3 / 597.5.
// Smaller ones lose alone: 2^20 17 M 167 / 171, 2^19 26 M 224 / 228, 60 tensors 288 / 297.  Stores alone, with that reader: 62 M step 645.7, 138 M 1577.6;
// loads alone 653.0, 1635.5.  The gradient read this way: 62 M step 535 / 551.
// Where the two are about even, columns of 2^8 behind a spectrum in memory and binary16 right above the line, it depends on what else is read: 2^16, four
// streams of 34.8 M samples, 8-bit codes of 10 % 174.9 / 168.2 and 242.2 / 250.2, of 50 % 169.2 / 163.0 and 233.9 / 244.0, of 90 % 177.9 / 166.9 and 241.8 / 245.0, 32-bit
// codes of 50 % 211.4 / 196.1 and 278.0 / 266.2, of 90 % 261.4 / 233.7 and 329.7 / 314.8; 45 M, 8 bits, 50 % 216.0 / 214.1 and 304.5 / 309.3; binary16, 2^16 33.6 M 89.3 /
// 84.2 and 155.4 / 160.2, 2^22 126.6 / 122.8 and 195.8 / 199.8, 2^20 94.6 / 85.1 and 158.9 / 160.2, 2^16 42 M 101.2 / 98.2 and 197.6 / 189.6.  A line of their own takes
// them longer in sum.
constexpr size_t kOnceBytes = (size_t)1 << 27;
template <int LOGN1, int LOGE, bool HALF, bool ONCE>
hipError_t inv_a_tiled(const float2* mid_f32, int logM, size_t C, float* out, size_t n, Tables t, bool aligned, float gain,
                  hipStream_t s, const uint32_t* only_if)
{
    const size_t lds = ((size_t)(1 << LOGE) + (1 << LOGN1)) * sizeof(float2);
    auto kern = k_inv_a<LOGN1, LOGE, HALF, ONCE>;
    auto* mid = reinterpret_cast<const typename Cx<HALF>::One*>(mid_f32);
    hipError_t e = set_lds(kern, lds);
    if (e != hipSuccess) return e;
    const size_t total = C * (((size_t)1 << (logM - LOGN1)) >> (LOGE - LOGN1));
    constexpr int glog = group_log(LOGE, LOGN1);
    const Grid g = grouped_grid(total >> glog, glog, most_wgs(LOGE, 512));
    FFTSP_LAUNCH(only_if ? "irfft_pass_a_standby" : "irfft_pass_a", kern, dim3(g.wgs), dim3(tile_lanes(LOGE)), lds, s, mid, logM, out,
                 n, t, aligned, (uint32_t)(total >> glog), g.per_wg, glog, gain, only_if);
    return hipGetLastError();
}

// Binary16 storage, rows of 2^8 and more: half the LDS per tile and a workgroup for each.  Whole calls in us, theta 0.3, 8 bits, fwd_b_tiled / this:
//   2^17 10 M samples 112 / 108.6, 42 M 287 / 278;  2^18 118.8 / 115.3, 275 / 264;  2^19 129 / 126, 303 / 294;  2^20 134 / 131, 62 M 442.5 / 434.5 (this
//   kernel 99 / 80);  2^21 25 M 227.5 / 227, 62 M 482.7 / 467.8;  2^22 33 M 302 / 297.6, 138 M 1119 / 1081;  2^16 45 M 306.7 / 311.8.  Senders, by tiles of 2^14: rows of
//   2^10, a workgroup a compute unit either way up to 256 of them, 128 (2^21) 54.9 / 57.1 and (2^22) 63.7 / 65.7, 192 65.0 / 65.1, 256 66.7 / 66.3 and 78.3 / 78.1, 384 86.3 /
//   83.5;  shorter rows from the first launches on that are not the short kernels': 2^17 128 42.4 / 41.0, 2^18 72 38.2 / 36.2, 2^19 128 45.0 / 44.5, 2^20 128 48.4 / 48.7, 192 55.9 /
//   54.7.
// Binary32 bins keep their persistent workgroups, which have a tile's loads on their way while they work on another: 2^16 45 M 364 / 381, 2^20 42 M
// 357 / 362.7, 2^22 67 M 661 / 674.
constexpr size_t kPairsForward10 = 192;  // tiles of 2^14 from which rows of 2^10 take it
template <int LOGN2>
hipError_t fwd_b_half(const float2* mid, int logM, size_t C, float2* spec, uint32_t sstride, Tables t, uint32_t* hist, float mid_scale, hipStream_t s)
{
    if constexpr (LOGN2 == 10)
        if (wide_tiles(C, logM) < kPairsForward10) return fwd_b_tiled<LOGN2, 14, true, true>(mid, logM, C, spec, sstride, t, hist, mid_scale, s, nullptr);
    constexpr size_t lds = HalfTile<LOGN2>::kLds + kHistLdsWords * sizeof(uint32_t);
    const auto kern = k_fwd_b_pairs<LOGN2, true>;
    const hipError_t e = set_lds(kern, lds);
    if (e != hipSuccess) return e;
    const size_t total = C << (logM - LOGN2 - 4);
    FFTSP_LAUNCH("rfft_pass_b", kern, dim3((unsigned)(8 * ((total + 7) / 8))), dim3(HalfTile<LOGN2>::NT), lds, s, reinterpret_cast<const uint32_t*>(mid), logM,
                 reinterpret_cast<uint32_t*>(spec), sstride, t, hist, (uint32_t)total, mid_scale);
    return hipGetLastError();
}
// the tile size by the rule at the top of the file
template <int LOGN2, bool CODEC, bool HALF>
hipError_t fwd_b(const float2* mid, int logM, size_t C, float2* spec, uint32_t sstride, Tables t, uint32_t* hist,
                 float mid_scale, hipStream_t s, const uint32_t* only_if = nullptr)
{
    if constexpr (LOGN2 >= kWideMin)
        if (wide_tiles(C, logM) >= kWideForward) return fwd_b_tiled<LOGN2, 14, CODEC, HALF>(mid, logM, C, spec, sstride, t, hist, mid_scale, s, only_if);
    return fwd_b_tiled<LOGN2, 13, CODEC, HALF>(mid, logM, C, spec, sstride, t, hist, mid_scale, s, only_if);
}
template <int LOGN2, bool PAIR, bool HALF>
hipError_t inv_b(const float2* spec, uint32_t sstride, int logM, size_t C, float2* mid, Tables t, float mid_scale,
                 hipStream_t s, const uint32_t* only_if = nullptr)
{
    if constexpr (LOGN2 >= kWideMin)
        if (wide_tiles(C, logM) >= kWideInverseB) return inv_b_tiled<LOGN2, 14, PAIR, HALF>(spec, sstride, logM, C, mid, t, mid_scale, s, only_if);
    return inv_b_tiled<LOGN2, 13, PAIR, HALF>(spec, sstride, logM, C, mid, t, mid_scale, s, only_if);
}
template <int LOGN1, int LOGE, bool HALF, bool ONCE>
hipError_t inv_a_halved(const float2* mid, int logM, size_t C, float* out, size_t n, Tables t, bool aligned, float gain, hipStream_t s, const uint32_t* only_if)
{
    using G = SplitInverse<LOGN1, LOGE>;
    const auto kern = k_inv_a_split<LOGN1, LOGE, HALF, ONCE>;
    const hipError_t e = set_lds(kern, G::kLds);
    if (e != hipSuccess) return e;
    const size_t total = C << (logM - LOGE);
    FFTSP_LAUNCH(only_if ? "irfft_pass_a_standby" : "irfft_pass_a", kern, dim3((unsigned)(8 * ((total + 7) / 8))), dim3(G::NT), G::kLds, s,
                 reinterpret_cast<const typename Cx<HALF>::One*>(mid), logM, out, n, t, aligned, (uint32_t)total, gain, only_if);
    return hipGetLastError();
}
template <int LOGN1, bool HALF>
hipError_t inv_a(const float2* mid, int logM, size_t C, float* out, size_t n, Tables t, bool aligned, float gain,
                 hipStream_t s, const uint32_t* only_if = nullptr)
{
    const size_t wide = wide_tiles(C, logM);
    const bool once = 4 * n >= kOnceBytes;
    auto persistent = [&](auto size, auto by) {
        return inv_a_tiled<LOGN1, decltype(size)::value, HALF, decltype(by)::value>(mid, logM, C, out, n, t, aligned, gain, s, only_if);
    };
    auto split = [&](auto size, auto by) {
        return inv_a_halved<LOGN1, decltype(size)::value, HALF, decltype(by)::value>(mid, logM, C, out, n, t, aligned, gain, s, only_if);
    };
    constexpr std::integral_constant<int, 13> small{};
    constexpr std::integral_constant<int, 14> large{};
    constexpr std::true_type by{};  // the caches: outputs with at least 2^10 large tiles
    constexpr std::false_type through{};
    static_assert(kOnceBytes >> 17 >= kSplitInverse10 && kOnceBytes >> 17 >= kSplitInverse11, "outputs that pass the caches by have large tiles");
    if constexpr (LOGN1 <= 8) {
        return once ? persistent(small, by) : persistent(small, through);
    } else if constexpr (LOGN1 == 9) {
        return once ? split(small, by) : split(small, through);
    } else if constexpr (LOGN1 == 10) {
        if (wide < kSplitInverse10) return split(small, through);
        return once ? split(large, by) : split(large, through);
    } else {
        if (once) return split(large, by);
        if (wide < kWideInverseA) return persistent(small, through);
        if constexpr (!HALF)
            if (wide >= kSplitInverse11) return persistent(large, through);
        return split(large, through);
    }
}

// The tensors come shortest first, so those whose rows ask for the larger tile are the last ones.  Beside shorter
// tensors they are a launch of their own, with two tails instead of one, 8 to 15 us, so the line lies higher than in uniform
// calls.  Senders and receivers in us, small / large tiles, of batches of 12 to 200 tensors of 10 to 2.4 M samples, not in
// the caches, by number of large tiles (of what the launch would hold): loses up to 1472 (of 2324) 458 / 476, 512 (of 1044)
// 206 / 210; 1536 (of 2048) 366 / 346.
constexpr size_t kWideInverseBBeside = 1536;
size_t launch_tiles(const LongBatch& b) { return (size_t)b.units << (kLongUnitLog - 14); }  // of 2^14 points
// The first of them, or count; alone, beside: large tiles that are enough.
template <typename Logs>
uint32_t first_wide(const LongBatch& b, Logs&& logs, size_t alone, size_t beside)
{
    uint32_t i = b.count;
    size_t tiles = 0;
    for (; i > 0 && logs(b.tab.t[i - 1].logM) >= kWideMin; --i) tiles += (size_t)1 << (b.tab.t[i - 1].logM - 14);
    return tiles >= (i == 0 ? alone : beside) ? i : b.count;
}
// tiles per workgroup (a power of two) that keep a launch over tensors [first, end) to about `most` workgroups
uint32_t long_run(const LongBatch& b, uint32_t first, uint32_t end, int loge, uint32_t most)
{
    size_t tiles = 0;
    for (uint32_t i = first; i < end; ++i) tiles += (size_t)1 << (b.tab.t[i].logM - loge);
    uint32_t run = 1;
    while (tiles / (2 * run) >= most) run *= 2;
    return run;
}
// pass(tile size, first tensor, end): those with small tiles, then the ones from `wide` on
template <typename Pass>
hipError_t by_tile_size(const LongBatch& b, uint32_t wide, Pass&& pass)
{
    hipError_t e = hipSuccess;
    if (wide > 0) e = pass(std::integral_constant<int, 13>{}, 0u, wide);
    if (e == hipSuccess && wide < b.count) e = pass(std::integral_constant<int, 14>{}, wide, b.count);
    return e;
}
// Up to how many tiles of 2^14 forward pass A has them as tiles of 2^13 whole in the LDS; with columns of 2^11 among them, which are 32 bytes wide then, as long as
// tiles of 2^14 would leave compute units idle.  Senders in us, in half of the LDS / whole, tensors of whole powers of two (and five samples less):
//   2^17 128 50.0 / 47.5 (50.1 / 47.8), 192 58.5 / 55.2;  2^18 128 50.5 / 47.4 (50.0 / 47.9), 256 68.7 / 65.6 (68.6 / 65.5), 384 87.4 / 86.2 (86.9 / 85.7);  2^19 128 53.4 / 50.9, 256 72.4 / 69.7
//   (72.0 / 69.1), 512 111 / 109 (109 / 110), 768 153.6 / 148.0 (153 / 150);  2^20 128 54.7 / 53.6 (55.4 / 53.9), 256 73.2 / 71.8 (74.1 / 72.8), 512 115 / 112 (119 / 115), 768 151 / 152 (154 / 156),
//   1536 253 / 256;  2^21 128 60.9 / 59.4 (61.2 / 59.9), 256 78.4 / 77.2 (79.5 / 77.9), 512 119.6 / 115.8 (122 / 118), 768 163.5 / 163.4 (167 / 167), 1024 199 / 197, 1536 277 / 279;
//   random sets 60 190 / 193, 100 205 / 210;  2^22 128 75.4 / 71.9 (75.2 / 71.8), beside shorter ones 130 78.9 / 76.8, 160 81.2 / 79.9, 192 84.1 / 82.1 and 80.2 /
//   77.8, 224 90.6 / 90.4, 256 89.7 / 90.0 (89.9 / 91.4) and 94.7 / 97.0, 384 120.1 / 122.2, 512 125.6 / 134.1.
// 256 are on the chip at once, and a few more a second round, which columns of 2^10 do not pay for: 2^21 and shorter ones 258 83.5 / 82.8, 264 85.2 / 88.9, 272 86.3 / 90.1 and 87.5 / 91.3, 288 90.8 /
// 92.4;  2^20 288 81.8 / 83.2, 320 84.0 / 87.5, 344 89.4 / 88.3, 352 90.6 / 89.6 and 99.9 / 98.5;  2^19 272 78.3 / 77.5, 304 81.8 / 80.5, 320 83.4 / 81.8;  2^18 264 74.2 / 73.9, 320 80.7 / 78.8.
bool whole_forward(const LongBatch& b)
{
    const size_t tiles = launch_tiles(b);
    const int columns = log_columns(b.tab.t[b.count - 1].logM);  // the longest come last
    if (columns > 10) return tiles < 256;
    return tiles <= 512 && (columns < 10 || tiles <= 256 || tiles >= 336);
}
// and up to how many, with rows of 2^10 and shorter ones, forward pass B has them as tiles of 2^13, one to a compute unit, where tiles of 2^14 would leave half of them
// idle.  Senders in us, tiles of 2^14 / this: 98 56.5 / 54.5, 104 57.0 / 55.3, 112 57.9 / 56.0, 128 60.7 / 58.8, 60.7 / 58.9 and 60.2 / 59.9, 130 63.8 / 63.9 and 76.2 / 74.8, 132 63.5 / 67.4 and
// 74.7 / 80.5, 136 64.0 / 67.3, 144 65.1 / 69.1, 160 66.4 / 70.1 and 68.2 / 69.5, 192 71.6 / 75.6.
constexpr size_t kFewBothRows = 130;
constexpr int kLongLogN = log_columns(kLongMax);  // the longest row or column
// LDS of a pass: the tile and the stage twiddles
constexpr size_t long_lds(int loge) { return ((size_t)(1 << loge) + (1 << kLongLogN)) * sizeof(float2); }
}  // namespace

int fft_pair_log(int logL)
{
    const int logM = logL - 1;
    return logM >= 14 ? (logM + 1) / 2 : 0;
}

hipError_t launch_rfft(const float* in, size_t n, int logL, size_t C, float* spec, uint32_t sstride, float2* mid,
                       Tables t, uint32_t* hist, uint32_t* zero_ptr, size_t zero_words, int pair_spec,
                       int* pair_log, hipStream_t s, const uint32_t* only_if)
{
    if (pair_log) *pair_log = 0;
    if (zero_words > 0xffffffffu) return hipErrorInvalidValue;
    if (!hist) zero_words = 0;
    const int logM = logL - 1;
    const bool aligned = aligned16(in);
    float2* sp = reinterpret_cast<float2*>(spec);
    if (logM < 15 || C * ((size_t)1 << (logM - 13)) > 0x7fffffffu) return hipErrorInvalidValue;
    // the codec stores its own spectrum in the paired order and wants the histogram; the stage-level entry point
    // wants neither
    if ((hist != nullptr) != (pair_spec != 0)) return hipErrorInvalidValue;
    const int logN1 = (logM + 1) / 2, logN2 = logM / 2;
    if (!only_if && short_forward(logM, C, 0)) {
        if (pair_log && pair_spec) *pair_log = logN1;
        return launch_short_rfft(in, n, logM, C, sp, sstride, mid, t, hist, zero_ptr, (uint32_t)zero_words, s);
    }
    hipError_t e;
#define FWD_A(p) fwd_a<p, false>(in, n, logM, C, mid, t, aligned, zero_ptr, zero_words, 1.0f, s, only_if)
    switch (logN1) {
        case 8: e = FWD_A(8); break;
        case 9: e = FWD_A(9); break;
        case 10: e = FWD_A(10); break;
        case 11: e = FWD_A(11); break;
        default: return hipErrorInvalidValue;
    }
#undef FWD_A
    if (e != hipSuccess) return e;
    if (pair_log && pair_spec) *pair_log = logN1;
    if (hist) {
        switch (logN2) {
            case 7: return fwd_b<7, true, false>(mid, logM, C, sp, sstride, t, hist, 1.0f, s, only_if);
            case 8: return fwd_b<8, true, false>(mid, logM, C, sp, sstride, t, hist, 1.0f, s, only_if);
            case 9: return fwd_b<9, true, false>(mid, logM, C, sp, sstride, t, hist, 1.0f, s, only_if);
            case 10: return fwd_b<10, true, false>(mid, logM, C, sp, sstride, t, hist, 1.0f, s, only_if);
            default: return hipErrorInvalidValue;
        }
    }
    switch (logN2) {
        case 7: return fwd_b<7, false, false>(mid, logM, C, sp, sstride, t, nullptr, 1.0f, s);
        case 8: return fwd_b<8, false, false>(mid, logM, C, sp, sstride, t, nullptr, 1.0f, s);
        case 9: return fwd_b<9, false, false>(mid, logM, C, sp, sstride, t, nullptr, 1.0f, s);
        case 10: return fwd_b<10, false, false>(mid, logM, C, sp, sstride, t, nullptr, 1.0f, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_irfft(const float* spec, uint32_t sstride, size_t n, int logL, size_t C, float* out, float2* mid,
                        Tables t, int pair_spec, float gain, hipStream_t s, const uint32_t* only_if)
{
    const int logM = logL - 1;
    const float2* sp = reinterpret_cast<const float2*>(spec);
    if (logM < 15 || C * ((size_t)1 << (logM - 13)) > 0x7fffffffu) return hipErrorInvalidValue;
    hipError_t e;
    if (!only_if && short_inverse(logM, C)) {
        e = launch_short_inverse_b(sp, sstride, logM, C, mid, t, pair_spec, s);
    } else if (pair_spec) {
        switch (logM / 2) {
            case 7: e = inv_b<7, true, false>(sp, sstride, logM, C, mid, t, 1.0f, s, only_if); break;
            case 8: e = inv_b<8, true, false>(sp, sstride, logM, C, mid, t, 1.0f, s, only_if); break;
            case 9: e = inv_b<9, true, false>(sp, sstride, logM, C, mid, t, 1.0f, s, only_if); break;
            case 10: e = inv_b<10, true, false>(sp, sstride, logM, C, mid, t, 1.0f, s, only_if); break;
            default: return hipErrorInvalidValue;
        }
    } else {
        switch (logM / 2) {
            case 7: e = inv_b<7, false, false>(sp, sstride, logM, C, mid, t, 1.0f, s); break;
            case 8: e = inv_b<8, false, false>(sp, sstride, logM, C, mid, t, 1.0f, s); break;
            case 9: e = inv_b<9, false, false>(sp, sstride, logM, C, mid, t, 1.0f, s); break;
            case 10: e = inv_b<10, false, false>(sp, sstride, logM, C, mid, t, 1.0f, s); break;
            default: return hipErrorInvalidValue;
        }
    }
    return e == hipSuccess ? launch_inverse_a(mid, logM, C, out, n, t, gain, 0, s, only_if) : e;
}

hipError_t launch_inverse_a(const float2* mid, int logM, size_t C, float* out, size_t n, Tables t, float gain, int half, hipStream_t s,
                            const uint32_t* only_if)
{
    if (half) gain *= half_lift(logM);
    if (!only_if && short_inverse(logM, C)) return launch_short_inverse_a(mid, logM, C, out, n, t, gain, half, s);
    const bool aligned = aligned16(out);
    auto run = [&](auto columns) {
        constexpr int LOGN1 = decltype(columns)::value;
        return half ? inv_a<LOGN1, true>(mid, logM, C, out, n, t, aligned, gain, s, only_if)
                    : inv_a<LOGN1, false>(mid, logM, C, out, n, t, aligned, gain, s, only_if);
    };
    switch ((logM + 1) / 2) {
        case 7: return half ? inv_a<7, true>(mid, logM, C, out, n, t, aligned, gain, s) : hipErrorInvalidValue;
        case 8: return run(std::integral_constant<int, 8>{});
        case 9: return run(std::integral_constant<int, 9>{});
        case 10: return run(std::integral_constant<int, 10>{});
        case 11: return run(std::integral_constant<int, 11>{});
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_rfft_long(const float* in, const LongBatch& b, float2* spec, float2* mid, Tables t, uint32_t* hist,
                            uint32_t* zero_ptr, size_t zero_words, hipStream_t s)
{
    if (b.count < 1 || b.count > (uint32_t)kMaxLongTensors || zero_words > 0xffffffffu) return hipErrorInvalidValue;
    if (short_forward(b)) return launch_short_rfft_long(in, b, spec, mid, t, hist, zero_ptr, (uint32_t)zero_words, s);
    LongStarts at;
    // What the XCDs begin further into a tensor each (stretches.h): three quarters of the launch are tensors of 128 tiles, or of 64 where all of it is on the chip at once.  Sender in us,
    // from the stretch's start / further: 20 of 2^20 131.1 / 133.4, 32 184.8 / 189.5, 48 of 2^19 148.9 / 150.1, 30 of 600 k 166.4 / 170.5;  eight of 2^20 (512 tiles) 74.6 / 72.1, twelve
    // 91.1 / 92.4;  beside shorter ones, of 2^21 32 and eight of 1 M 446 / 437, and 24 of 300 k 467 / 462, 16 and 24 254.2 / 254.9, random sets 292.7 / 297.1 and 265.3 / 267.7.
    auto step_of = [&](uint32_t total, int loge) {
        const uint32_t least = loge == kTileFA && total <= 512u ? 64u : 128u;
        uint32_t tiles = 0;  // of those
        for (uint32_t i = b.count; i > 0 && power_tiles(b.tab.t[i - 1].logM, loge) >= least; --i) tiles += power_tiles(b.tab.t[i - 1].logM, loge);
        return 4u * tiles >= 3u * total ? kTurnStep : 0u;
    };
    auto whole = [&]() {
        const hipError_t err = set_lds(k_fwd_a_long, long_lds(kTileFA));
        if (err != hipSuccess) return err;
        const uint32_t total = long_starts(b, 0, b.count, &at, [](int logM) { return power_tiles(logM, kTileFA); });
        FFTSP_LAUNCH("rfft_pass_a", k_fwd_a_long, dim3(stretch_places(total)), dim3(tile_lanes(kTileFA)), long_lds(kTileFA), s, in, mid, t, total, step_of(total, kTileFA),
                     zero_ptr, (uint32_t)zero_words, b.tab, at);
        return hipGetLastError();
    };
    auto pass_a = [&](auto size) {
        constexpr int TOP = decltype(size)::value;
        constexpr size_t lds = SplitTile<TOP == 14 ? 11 : 10, TOP>::kLds;
        const hipError_t err = set_lds(k_fwd_a_split_long<TOP>, lds);
        if (err != hipSuccess) return err;
        const uint32_t total = long_starts(b, 0, b.count, &at, [](int logM) { return power_tiles(logM, TOP); });
        FFTSP_LAUNCH("rfft_pass_a", k_fwd_a_split_long<TOP>, dim3((total + 7) / 8 * 8), dim3(tile_lanes(TOP)), lds, s, in, mid, t, total, step_of(total, TOP), zero_ptr,
                     (uint32_t)zero_words, b.tab, at);
        return hipGetLastError();
    };
    const bool narrow = log_columns(b.tab.t[b.count - 1].logM) <= 10;
    const hipError_t e = whole_forward(b) ? whole() : narrow ? pass_a(std::integral_constant<int, 13>{}) : pass_a(std::integral_constant<int, 14>{});
    return e == hipSuccess ? launch_rfft_b_long(b, spec, mid, t, hist, s) : e;
}

hipError_t launch_rfft_b_long(const LongBatch& b, float2* spec, const float2* mid, Tables t, uint32_t* hist, hipStream_t s)
{
    if (b.count < 1 || b.count > (uint32_t)kMaxLongTensors) return hipErrorInvalidValue;
    if (short_forward(b)) return launch_short_rfft_b_long(b, spec, mid, t, hist, s);
    LongStarts at;
    uint32_t tall = b.count;  // the first with rows of 2^10: the longest come last
    while (tall > 0 && log_rows(b.tab.t[tall - 1].logM) >= 10) --tall;
    // One launch, whatever the rows' lengths.  From 131 tiles on persistent workgroups (k_fwd_b_long) pay for their runs of tiles in most launch sets, and a launch of their
    // own for rows of 2^10 for a tail.  Sender and receiver in us, before (k_fwd_b_long<13> where rows of 2^10 were among few tiles, a launch for either from
    // 512 large tiles on) / this: random sets of 30 248 / 236.5, 40 279 / 269, 60 272.5 / 264, 100 471 / 450,
    // 200 746 / 723, 40 of 1 M and four of 2^21 470 / 445, 30 and ten 502 / 473, ten of 500 k and sixteen 371 / 364, 55 of 70 k and one 158 / 151.  Senders, a launch of persistent workgroups for rows of 2^10 beside one for the others / one
    // for all: one of 2^16 and eight of 2^21 130.3 / 124.2, 24 287 / 268, 32 420 / 412, 48 596 / 586, and eight of 2^22 236.5 / 230.5, 16 454 / 434.
    // Rows of 2^10 alone it gains about as often as it loses: 2^21 four 122 / 127, eight 174 / 173, twelve 243 / 238, 24 431 / 422, 32 565 / 581;  2^22 eight
    // 314 / 321, sixteen 579 / 586.
    auto pairs = [&](auto size) {
        constexpr int TOP = decltype(size)::value;
        const hipError_t err = set_lds(k_fwd_b_pairs_long<TOP>, kPairsLds<TOP>);
        if (err != hipSuccess) return err;
        const uint32_t total = long_starts(b, 0, b.count, &at, [](int logM) { return power_tiles(logM, TOP + 4); });
        const uint32_t few = TOP == 10 ? few_apart(total, at.at[tall]) : 0u;
        FFTSP_LAUNCH("rfft_pass_b", k_fwd_b_pairs_long<TOP>, dim3(stretch_places(total, few)), dim3(HalfTile<TOP>::NT), kPairsLds<TOP>, s, mid, spec, t, hist,
                     total, few, b.tab, at);
        return hipGetLastError();
    };
    if (tall == b.count) return pairs(std::integral_constant<int, 9>{});
    if (tall > 0 && launch_tiles(b) > kFewBothRows) return pairs(std::integral_constant<int, 10>{});
    auto runs = [&](auto size) {
        constexpr int LOGE = decltype(size)::value;
        const size_t lds = long_lds(LOGE) + kHistLdsWords * sizeof(uint32_t);
        const hipError_t err = set_lds(k_fwd_b_long<LOGE>, lds);
        if (err != hipSuccess) return err;
        const uint32_t per = long_run(b, 0, b.count, LOGE, most_wgs(LOGE, 512));
        const uint32_t g = long_starts(b, 0, b.count, &at, [&](int logM) {
            const uint32_t tiles = power_tiles(logM, LOGE);
            return tiles > per ? tiles / per : 1u;
        });
        FFTSP_LAUNCH("rfft_pass_b", k_fwd_b_long<LOGE>, dim3(g), dim3(tile_lanes(LOGE)), lds, s, mid, spec, t, hist, per, b.tab, at);
        return hipGetLastError();
    };
    return tall > 0 ? runs(std::integral_constant<int, 13>{}) : runs(std::integral_constant<int, kTallTile>{});
}

hipError_t launch_irfft_long(const float2* spec, const LongBatch& b, float* out, float2* mid, Tables t, hipStream_t s)
{
    if (b.count < 1 || b.count > (uint32_t)kMaxLongTensors) return hipErrorInvalidValue;
    hipError_t e;
    if (short_inverse(b)) {
        e = launch_short_inverse_b_long(spec, b, mid, t, s);
    } else {
        LongStarts at;
        const uint32_t wide = first_wide(b, log_rows, kWideInverseB, kWideInverseBBeside);
        e = by_tile_size(b, wide, [&](auto size, uint32_t first, uint32_t end) {
            constexpr int LOGE = decltype(size)::value;
            const hipError_t err = set_lds(k_inv_b_long<LOGE>, long_lds(LOGE));
            if (err != hipSuccess) return err;
            const uint32_t per = long_run(b, first, end, LOGE, most_wgs(LOGE, 1536));
            const uint32_t g = long_starts(b, first, end, &at, [&](int logM) {
                const uint32_t tiles = power_tiles(logM, LOGE);
                return tiles > per ? tiles / per : 1u;
            });
            FFTSP_LAUNCH("irfft_pass_b", k_inv_b_long<LOGE>, dim3(g), dim3(tile_lanes(LOGE)), long_lds(LOGE), s, spec, mid, t, per, b.tab, at);
            return hipGetLastError();
        });
    }
    return e == hipSuccess ? launch_inverse_a_long(mid, b, out, t, s) : e;
}

hipError_t launch_inverse_a_long(const float2* mid, const LongBatch& b, float* out, Tables t, hipStream_t s)
{
    if (b.count < 1 || b.count > (uint32_t)kMaxLongTensors) return hipErrorInvalidValue;
    if (short_inverse(b)) return launch_short_inverse_a_long(b, out, mid, t, s);
    const bool aligned = aligned16(out);
    LongStarts at;
    // Tiles of 2^13 as in uniform calls; launches with columns of 2^11 have them beside tiles of 2^14, two to a workgroup.  Receivers in us,
    // persistent (a launch for each tile size) / this: ResNet-50's 161 tensors 159 / 136, 150 of 10 to 2.4 M samples 224 / 161, 100 164 / 134, 60 82 / 79 and (longer)
    // 124 / 101.5, 48 of 2^19 89 / 79, of 2^19 - 1 107 / 83, 18 of 2^20 78 / 68, 30 116 / 103, 60 (tiles of 2^14) 266.5 / 210, of 2^20 - 3 328 / 266, 120 of 2^18 138.5 / 115.5,
    // 5 of 3 M 100 / 85, of 3 000 001 117 / 89.5, 180 of 2^16 63.6 / 63.7.
    const bool small = log_columns(b.tab.t[b.count - 1].logM) <= (launch_tiles(b) < kSplitInverse10 ? 10 : 9);
    auto run = [&](auto size) {
        constexpr int TOP = decltype(size)::value;
        constexpr size_t lds = SplitInverse<TOP == 14 ? 11 : 10, TOP>::kLds;
        const hipError_t err = set_lds(k_inv_a_split_long<TOP>, lds);
        if (err != hipSuccess) return err;
        const uint32_t total = long_starts(b, 0, b.count, &at, [](int logM) { return power_tiles(logM, TOP); });
        FFTSP_LAUNCH("irfft_pass_a", k_inv_a_split_long<TOP>, dim3((total + 7) / 8 * 8), dim3(tile_lanes(TOP)), lds, s, mid, out, t, aligned, total, b.tab, at);
        return hipGetLastError();
    };
    return small ? run(std::integral_constant<int, 13>{}) : run(std::integral_constant<int, 14>{});
}

// Half-precision variant (two-pass sizes, the codec's own buffers): the same four kernels with the intermediate
// and the spectrum stored as binary16 pairs.  in_scale (a power of two) multiplies the samples on the way in;
// the receiver divides through `gain`.
hipError_t launch_rfft_half(const float* in, size_t n, int logL, size_t C, void* spec, uint32_t sstride, void* mid,
                            Tables t, uint32_t* hist, uint32_t* zero_ptr, size_t zero_words, float in_scale,
                            int* pair_log, hipStream_t s)
{
    const int logM = logL - 1;
    if (logM < 14 || !hist || zero_words > 0xffffffffu) return hipErrorInvalidValue;
    if (C * ((size_t)1 << (logM - 13)) > 0x7fffffffu) return hipErrorInvalidValue;
    const bool aligned = aligned16(in);
    float2* sp = static_cast<float2*>(spec);
    float2* md = static_cast<float2*>(mid);
    const int logN1 = (logM + 1) / 2, logN2 = logM / 2;
    hipError_t e;
    const float lift = half_lift(logM);
    if (short_forward(logM, C, 1)) {
        *pair_log = logN1;
        return launch_short_rfft_half(in, n, logM, C, sp, sstride, md, t, hist, zero_ptr, (uint32_t)zero_words, in_scale * lift, 1.0f / lift, s);
    }
#define FWD_A(p) \
    fwd_a<p, true>(in, n, logM, C, md, t, aligned, zero_ptr, (uint32_t)zero_words, in_scale * lift, s)
    switch (logN1) {
        case 7: e = FWD_A(7); break;
        case 8: e = FWD_A(8); break;
        case 9: e = FWD_A(9); break;
        case 10: e = FWD_A(10); break;
        case 11: e = FWD_A(11); break;
        default: return hipErrorInvalidValue;
    }
#undef FWD_A
    if (e != hipSuccess) return e;
    *pair_log = logN1;
    switch (logN2) {
        case 7: return fwd_b<7, true, true>(md, logM, C, sp, sstride, t, hist, 1.0f / lift, s);
        case 8: return fwd_b_half<8>(md, logM, C, sp, sstride, t, hist, 1.0f / lift, s);
        case 9: return fwd_b_half<9>(md, logM, C, sp, sstride, t, hist, 1.0f / lift, s);
        case 10: return fwd_b_half<10>(md, logM, C, sp, sstride, t, hist, 1.0f / lift, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_irfft_half(const void* spec, uint32_t sstride, size_t n, int logL, size_t C, float* out, void* mid,
                             Tables t, float gain, hipStream_t s)
{
    const int logM = logL - 1;
    if (logM < 14) return hipErrorInvalidValue;
    if (C * ((size_t)1 << (logM - 13)) > 0x7fffffffu) return hipErrorInvalidValue;
    const float2* sp = static_cast<const float2*>(spec);
    float2* md = static_cast<float2*>(mid);
    const float lower = 1.0f / half_lift(logM);
    hipError_t e;
    if (short_inverse(logM, C)) {
        e = launch_short_inverse_b_half(sp, sstride, logM, C, md, t, lower, s);
    } else {
        switch (logM / 2) {
            case 7: e = inv_b<7, true, true>(sp, sstride, logM, C, md, t, lower, s); break;
            case 8: e = inv_b<8, true, true>(sp, sstride, logM, C, md, t, lower, s); break;
            case 9: e = inv_b<9, true, true>(sp, sstride, logM, C, md, t, lower, s); break;
            case 10: e = inv_b<10, true, true>(sp, sstride, logM, C, md, t, lower, s); break;
            default: return hipErrorInvalidValue;
        }
    }
    return e == hipSuccess ? launch_inverse_a(md, logM, C, out, n, t, gain, 1, s) : e;
}

}  // namespace fftsp

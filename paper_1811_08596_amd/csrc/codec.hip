// Selection, quantization, packing and their inverses for gfx950.
//
// Follows arXiv 1811.08596: Sec. 3.1.1 (keep the largest-magnitude frequency
// components, zero the rest), Sec. 3.2 (status bitmap -> prefix sum -> dense
// vector) and Sec. 3.2.1 / Algorithm 1 (offset-based N-bit float).
//
// Selection is an exact radix select on the 31-bit key
//     key = bits( fma(re, re, im*im) )        (binary32, one product rounded, then one fused step)
// so it is integer work: a 12-bit histogram of the top key bits per chunk finds
// the bucket that holds the k-th largest key; bins in higher buckets are kept
// outright, bins in that bucket ("candidates") are written out tile by tile in
// bin order, and one workgroup per chunk finishes the select on the candidates
// (two more digits), resolves ties by lowest bin index, scans the per-tile
// survivor counts and finds the survivors' largest component, which fixes eps
// (pbase) of Algorithm 1.  A last pass flags, ranks (wave ballots + popcounts),
// quantizes and bit-packs.
#include "codec_core.h"
#include "sample.h"

#include <algorithm>
#include <type_traits>

namespace fftsp {
namespace {

constexpr int NT = kTileThreads;     // 256 lanes = 4 waves
constexpr int ROWS = 8;              // rows of 64 bins per wave
constexpr int WAVE_BINS = ROWS * 64; // 512
static_assert(kTile == 4 * WAVE_BINS, "tile geometry");

// The tile at X to LDS, as whole 16-byte pieces where it is complete and X aligned.  A tile is contiguous in the spectrum
// buffer in either bin order (paired runs are tile-aligned).
template <typename T>
__device__ __forceinline__ void tile_to_lds(const T* __restrict__ X, uint32_t count, bool aligned, T* stage, int tid)
{
    constexpr int PER = 16 / (int)sizeof(T);
    if (count == (uint32_t)kTile && aligned) {
        const float4* src = reinterpret_cast<const float4*>(X);
        float4* dst = reinterpret_cast<float4*>(stage);
#pragma unroll
        for (int i = 0; i < kTile / PER / kTileThreads; ++i) dst[tid + i * kTileThreads] = src[tid + i * kTileThreads];
    } else {
        for (uint32_t i = tid; i < count; i += kTileThreads) stage[i] = X[i];
    }
}

// A wave's 512 units of the tile at X (whose first `count` units exist), in memory or in LDS: row r of 64 starts at the
// tile's unit row0 + 64 r.  In paired order a row's slots are two apart, upwards in the lower half of its run and downwards
// in the upper one, whose first bin N1/2 sits at position 1, off that line (a run has at least 128 positions and a tile
// is whole runs, so a row lies in one half of one run).
template <typename T, typename E>
__device__ __forceinline__ void load_units(const T* __restrict__ X, uint32_t row0, uint32_t count, int lane, int pair_log,
                                           E (&z)[ROWS])
{
    T raw[ROWS];
    if (count < (uint32_t)kTile) {  // the end of a chunk: units that do not exist read its last one, or count as zeros
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint32_t j = row0 + (uint32_t)(r * 64 + lane);
            const bool in = j < count;
            const uint32_t at = count ? spec_index(in ? j : count - 1u, pair_log) : 0u;
            raw[r] = count ? X[at] : T();
            if constexpr (std::is_same_v<T, float>) raw[r] = in ? raw[r] : 0.f;
        }
    } else if (pair_log == 0) {
        const T* p = X + row0 + lane;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) raw[r] = p[r * 64];
    } else if (pair_log >= 10) {
        const uint32_t N1 = 1u << pair_log, half = N1 / 2, run = row0 & ~(N1 - 1u), k1 = row0 - run;
        if (k1 < half) {
            const T* p = X + run + 2u * (k1 + (uint32_t)lane);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) raw[r] = p[r * 128];
        } else {
            const uint32_t last = run + 2u * (N1 - k1 - 64u * (ROWS - 1) - (uint32_t)lane) + 1u;  // row ROWS-1
            const T* p = X + last;
#pragma unroll
            for (int r = 1; r < ROWS; ++r) raw[r] = p[(ROWS - 1 - r) * 128];
            raw[0] = X[k1 == half && lane == 0 ? run + 1u : last + 128u * (ROWS - 1)];
        }
    } else {
        const uint32_t N1 = 1u << pair_log, half = N1 / 2;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint32_t row = row0 + (uint32_t)r * 64u, run = row & ~(N1 - 1u), k1 = row - run;
            const uint32_t slot = k1 < half ? run + 2u * (k1 + (uint32_t)lane) : run + 2u * (N1 - k1 - (uint32_t)lane) + 1u;
            raw[r] = X[k1 == half && lane == 0 ? run + 1u : slot];
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        if constexpr (std::is_same_v<T, float>)
            z[r] = raw[r];
        else
            z[r] = cx_load(raw[r]);
    }
}
// units of the tile at tbase that hold data (samples: the last chunk may end early, the rest counts as zeros)
template <bool REAL>
__device__ __forceinline__ uint32_t units_in_tile(size_t n, size_t c, uint32_t B, uint32_t tbase)
{
    const uint32_t end = present_of<REAL>(n, c, B);
    return end <= tbase ? 0u : (end - tbase < (uint32_t)kTile ? end - tbase : (uint32_t)kTile);
}
// lanes of the row of 64 units starting at unit j of a chunk of B that exist
__device__ __forceinline__ uint64_t row_mask(uint32_t j, uint32_t B)
{
    return j + 64u <= B ? ~0ull : (j >= B ? 0ull : (1ull << (B - j)) - 1ull);
}

__global__ void k_zero_u32(uint32_t* p, size_t count)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0u;
}

// ------------------------------------------------------------- histogram ----
constexpr int HIST_TILES = 4;  // tiles per workgroup

__global__ __launch_bounds__(NT) void k_hist(const float2* __restrict__ spec, uint32_t sstride, int pair_log, uint32_t B,
                                             uint32_t groups, uint32_t* __restrict__ hist)
{
    __shared__ uint32_t h[kHistBins];
    const int tid = threadIdx.x;
    const size_t c = blockIdx.x / groups;
    const uint32_t base = (blockIdx.x % groups) * (HIST_TILES * kTile);
    for (int i = tid; i < kHistBins; i += NT) h[i] = 0u;
    __syncthreads();
    const float2* X = spec + c * (size_t)sstride;
#pragma unroll 4
    for (int i = tid; i < HIST_TILES * kTile; i += NT) {
        const uint32_t j = base + i;
        if (j < B) atomicAdd(&h[key_of(X[spec_index(j, pair_log)]) >> kKeyShift], 1u);
    }
    __syncthreads();
    uint32_t* g = hist + c * kHistBins;
    for (int i = tid; i < kHistBins; i += NT) {
        const uint32_t v = h[i];
        if (v) atomicAdd(&g[i], v);
    }
}

// Time domain: the same histogram over the samples' |x| patterns, as a kernel of its own because it is the first
// and largest pass of that path.  Gradients crowd into a few dozen of the buckets (16 per binade), so plain LDS
// counters serialise; here every lane adds into one of kHistCopies copies chosen by its lane id, the copies are
// skewed by one bank each, and a counter is a 16-bit half of a word (a copy receives at most 8192 keys).
// Measured on 62 M samples: 2 copies x 8 tiles 76 us; 1 x 8: 82; 4 x 8: 85; 2 x 4: 92; 2 x 16: 95; 8 x 16: 126
// (more LDS per workgroup costs residency, shorter stretches pay the flush more often).  The first loads go out before the counters are
// cleared, and the flush adds to neighbouring counters: 77.5 -> 73.4; 512 lanes on 16 tiles 81, 1024 on 32 84.
constexpr int kHistCopies = 2;
constexpr int kHistSampleTiles = 8;  // tiles of 2048 samples per workgroup
constexpr int kHistCopyWords = kHistBins / 2 + 1;
static_assert(kHistSampleTiles * kTile / kHistCopies < 65536, "16-bit counters");

__global__ __launch_bounds__(NT) void k_hist_samples(const float* __restrict__ in, uint32_t L, uint32_t groups,
                                                     uint32_t* __restrict__ hist, size_t n)
{
    __shared__ __align__(16) uint32_t h[(kHistCopies * kHistCopyWords + 3) / 4 * 4];
    const int tid = threadIdx.x;
    const size_t c = blockIdx.x / groups;
    const uint32_t base = (blockIdx.x % groups) * (uint32_t)(kHistSampleTiles * kTile);
    const float* X = in + c * (size_t)L;
    const uint32_t present = present_of<true>(n, c, L);
    const uint32_t count = L - base < (uint32_t)(kHistSampleTiles * kTile) ? L - base : (uint32_t)(kHistSampleTiles * kTile);
    uint32_t* mine = h + (tid & (kHistCopies - 1)) * kHistCopyWords;
    auto add = [&](float x) __attribute__((always_inline)) {
        const uint32_t b = key_of(x) >> kKeyShift;
        atomicAdd(&mine[b >> 1], 1u << (16u * (b & 1u)));
    };
    auto clear = [&]() __attribute__((always_inline)) {
        for (int i = tid; i < (int)(sizeof(h) / 16); i += NT) reinterpret_cast<uint4*>(h)[i] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
    };
    constexpr int PER = kHistSampleTiles * kTile / 4 / NT, STEP = 4;  // float4 of a lane; in flight beside the ones being counted
    const float4* X4 = reinterpret_cast<const float4*>(X + base);  // chunks start on multiples of 32 samples of a 16-byte aligned gradient
    if (count == (uint32_t)(kHistSampleTiles * kTile) && base + count <= present) {
        float4 v[2][STEP];
        auto load = [&](int g) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < STEP; ++i) v[g & 1][i] = X4[tid + (g * STEP + i) * NT];
        };
        load(0);
        clear();
#pragma unroll
        for (int g = 0; g < PER / STEP; ++g) {
            if (g + 1 < PER / STEP) load(g + 1);
#pragma unroll
            for (int i = 0; i < STEP; ++i) {
                add(v[g & 1][i].x);
                add(v[g & 1][i].y);
                add(v[g & 1][i].z);
                add(v[g & 1][i].w);
            }
        }
    } else if (base + count <= present) {
        clear();
        for (uint32_t i = tid; i < count / 4u; i += NT) {
            const float4 v = X4[i];
            add(v.x);
            add(v.y);
            add(v.z);
            add(v.w);
        }
    } else {  // the gradient ends inside this stretch or before it: what lies past its end counts as zeros
        clear();
        const uint32_t here = present > base ? present - base : 0u;
        for (uint32_t i = tid; i < here; i += NT) add(X[base + i]);
        if (tid == 0) atomicAdd(&mine[0], count - here);  // into the low half: fewer than 2^16
    }
    __syncthreads();
    // neighbouring lanes add to neighbouring counters: a row of 64 is then one request and not two of every other word
    uint32_t* g = hist + c * kHistBins;
#pragma unroll 4
    for (int i = tid; i < kHistBins; i += NT) {
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kHistCopies; ++k) sum += h[k * kHistCopyWords + (i >> 1)] >> (16 * (i & 1)) & 0xFFFFu;
        if (sum) atomicAdd(&g[i], sum);
    }
}

// inclusive scan over the NW waves of a workgroup; tmp has NW entries
template <int NW>
__device__ __forceinline__ uint32_t block_scan_incl(uint32_t v, uint32_t* tmp)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t x = wave_scan_incl(v);
    if (lane == 63) tmp[wave] = x;
    __syncthreads();
    uint32_t add = 0;
#pragma unroll
    for (int w = 0; w < NW - 1; ++w) add += w < wave ? tmp[w] : 0u;
    __syncthreads();
    return x + add;
}

// What a workgroup of the codec kernels works on: a chunk and one of its tiles.  Uniform launches: all chunks are alike, and
// everything about them but the index comes with the launch.  Tables (per-tensor calls): looked up.
struct Place {
    uint32_t chunk, tile;        // tile: number within the chunk
    uint32_t B, Tn, W, k;        // bins, tiles, bitmap words, kept bins of the chunk
    uint32_t tile0, group0;      // the chunk's first tile and its first group of bitmap words, in the launch's work areas
    size_t spec, record, S;      // its spectrum (in bins), its record (byte offset and size)
    uint32_t word3;
    int pair_log;
};
struct Shape {  // of a uniform launch
    uint32_t B, Tn, W, k, sstride, word3;
    size_t S;
    int pair_log;
};
template <bool TABLE>
__device__ __forceinline__ Place place_of(const Shape& u, const TableArg<TABLE>& tab, uint32_t chunk, uint32_t tile)
{
    if constexpr (TABLE) {
        const LongTensor& x = tab.t.t[chunk];
        const uint32_t M = 1u << x.logM;
        return Place{chunk, tile, M + 1u, M / (uint32_t)kTile + 1u, M / 32u + 1u, x.kept, long_tile(x, chunk), long_group(x, chunk),
                     long_spec(x, chunk), (size_t)x.roff, x.stride, 2u * M, long_pair_log(x)};
    } else {
        const uint32_t G = (u.W + 15u) / 16u;
        return Place{chunk, tile, u.B, u.Tn, u.W, u.k, chunk * u.Tn, chunk * G, chunk * (size_t)u.sstride, chunk * u.S, u.S,
                     u.word3, u.pair_log};
    }
}
// a workgroup per tile
template <bool TABLE>
__device__ __forceinline__ Place place_of_tile(const Shape& u, const TableArg<TABLE>& tab, uint32_t tile = blockIdx.x)
{
    if constexpr (TABLE) {
        const LongShare share = long_share(tab.t.tiles, tile);
        return place_of<TABLE>(u, tab, share.tensor, share.blk);
    } else {
        return place_of<TABLE>(u, tab, tile / u.Tn, tile % u.Tn);
    }
}

// The bucket b* holding the k-th largest key of a chunk, and how many of its bins are still needed; by a whole workgroup.
struct Bucket {
    uint32_t star, need;
};
__device__ __forceinline__ Bucket find_bucket(const uint32_t* __restrict__ hist, uint32_t k)
{
    __shared__ uint32_t tmp[NT / 64], found[2];
    const int tid = threadIdx.x;
    constexpr int PER = kHistBins / NT;  // 16 buckets per lane, lane t owns the buckets counted from the top
    uint32_t loc[PER];
    const uint32_t top = kHistBins - 1 - tid * PER;  // highest bucket of this lane
#pragma unroll
    for (int i = 0; i < PER; i += 4) {
        const uint4 v = *reinterpret_cast<const uint4*>(hist + (top - i - 3));
        loc[i] = v.w;
        loc[i + 1] = v.z;
        loc[i + 2] = v.y;
        loc[i + 3] = v.x;
    }
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) s += loc[i];
    // The histogram counts every bin of the chunk, so some bucket always qualifies unless k is 0 (then nothing is kept);
    // should it ever not (fewer than k bins counted), the result is still defined.
    if (tid == 0) {
        found[0] = k == 0 ? (uint32_t)kHistBins : 0u;
        found[1] = 0;
    }
    uint32_t run = block_scan_incl<NT / 64>(s, tmp) - s;  // bins in buckets above this lane's range
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (run < k && run + loc[i] >= k) {
            found[0] = top - i;
            found[1] = k - run;
        }
        run += loc[i];
    }
    __syncthreads();
    return Bucket{found[0], found[1]};
}

template <bool TABLE>
__global__ __launch_bounds__(NT) void k_find_bucket(const uint32_t* __restrict__ hist, Shape u, uint32_t* __restrict__ sel,
                                                    TableArg<TABLE> tab)
{
    const size_t c = blockIdx.x;
    const Bucket b = find_bucket(hist + c * kHistBins, place_of<TABLE>(u, tab, blockIdx.x, 0u).k);
    if (threadIdx.x == 0) *reinterpret_cast<uint2*>(sel + c * 8) = make_uint2(b.star, b.need);
}

// Tiles of a chunk whose candidates k_resolve keeps in registers.  Longer chunks go through k_count_digit and k_mark before it, and
// where some of a launch do, so do those of more than kFewTiles beside them.
constexpr uint32_t kKeptTiles = 513, kFewTiles = 288;
// Tiles of a chunk up to which k_emit may do k_resolve's work.
constexpr uint32_t kMergedTiles = 72;

// a digit d, counted for the lanes that want it
__device__ __forceinline__ void count_digit(uint32_t* h, bool hit, uint32_t d, bool run_likely, int lane, uint32_t weight)
{
    if (run_likely) {
        const uint64_t act = __ballot(hit);
        if (!act) return;
        // a row whose keys share the digit (a run of equal values, e.g. zeros) is one atomic
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, __ffsll((unsigned long long)act) - 1);
        if (__ballot(hit && d == d0) == act) {
            if (lane == 0) atomicAdd(&h[d0], (uint32_t)__popcll(act) * weight);
            return;
        }
    }
    if (hit) atomicAdd(&h[d], weight);
}
// ---------------------------------------------------------------- sample ----
// Time domain, chunks of up to kKeptTiles tiles: the samples are not counted.  A workgroup per chunk looks at 2^15 of them and says between which
// two keys the k-th largest lies, so widely that it all but always does; k_collect then takes those above as kept and those between as
// candidates, and k_resolve, which knows how many are above, sees whether the k-th largest is among the candidates.  Where it is not, it selects
// from the samples themselves (select_samples): the result is exact whatever was sampled.
//
// The sample: stretches of eight or sixteen neighbours (sample_stretch), one from each equal part of the chunk, at a place in it that a hash of its number
// says, so that no period of the gradient's layout is met again and again.  Neighbours are alike in a gradient, so how far the sample's ranks are off
// is taken from the stretches: half the squared differences between one's count above the estimate and the next one's, which is what independent
// samples' ranks vary by too where there is no likeness (sample_variance).  Four and a half of these standard deviations either side: 38 candidates to a
// tile of 2048 at 15 % kept, where a bucket of the histogram has 10 to 40, and one chunk in 150000 whose threshold lies outside.  More than 128 to a tile are
// slow: with five and a half, and stretches of sixteen, 62 M samples in chunks of 2^20, 15 % kept, took 133.7 us, rows of 64 with a scale each 166, 50 % of a sine 351.
//
// Zeros are never candidates: a gradient can be half zeros (a rectifier's), and a window that reached them would have k_collect write most of
// the chunk.  Where the window's lower end is the smallest key above zero and the candidates do not have the threshold, it is zero.
//
// Bound by latency: one trip to memory, behind what the call before has left to write, and the barriers of three scans.  Sixty chunks of 2^20:
// 22 us, where clearing the histograms, counting 62 M samples and finding the buckets took 83; k_collect, which then is the first to read all of the
// gradient, 42 -> 59, k_resolve 21 -> 30.
constexpr int kSampleLanes = 1024, kSampleLoads = 8;
static_assert(4 * kSampleLanes * kSampleLoads == kSamples, "four samples a load");
// SHARE: log2 of the lanes that share a stretch
template <int SHARE>
__global__ __launch_bounds__(kSampleLanes) void k_sample(const float* __restrict__ in, uint32_t L, uint32_t k, size_t n, uint32_t* __restrict__ sel,
                                                        uint32_t* __restrict__ ctl)
{
    constexpr int NW = kSampleLanes / 64;
    __shared__ __align__(16) uint32_t h[kHistBins];
    __shared__ uint32_t fine[kHist2Bins], sums[3][NW], edge[6];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t c = blockIdx.x;
    if (c == 0 && tid < (int)(kControlBytes / 4)) ctl[tid] = 0u;
    if (k == 0) {  // nothing is kept, and nothing is a candidate
        if (tid == 0) *reinterpret_cast<uint2*>(sel + c * 8) = make_uint2(0xFFFFFFFFu, 0xFFFFFFFFu);
        return;
    }
    const float* X = in + c * (size_t)L;
    const uint32_t present = present_of<true>(n, c, L), slots = L / kSamples;
    uint32_t key[4 * kSampleLoads];
#pragma unroll
    for (int j = 0; j < kSampleLoads; ++j) {
        const uint32_t g = (uint32_t)(j * (kSampleLanes >> SHARE) + (tid >> SHARE)), at = (4u << SHARE) * (g * slots + sample_slot(g, slots)) + 4u * ((uint32_t)tid & ((1u << SHARE) - 1u));
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (at + 4u <= present) {
            v = *reinterpret_cast<const float4*>(X + at);
        } else if (at < present) {
            v.x = X[at];
            if (at + 1u < present) v.y = X[at + 1u];
            if (at + 2u < present) v.z = X[at + 2u];
        }
        key[4 * j] = key_of(v.x);
        key[4 * j + 1] = key_of(v.y);
        key[4 * j + 2] = key_of(v.z);
        key[4 * j + 3] = key_of(v.w);
    }
    reinterpret_cast<uint4*>(h)[tid] = make_uint4(0u, 0u, 0u, 0u);
    static_assert(kHistBins == 4 * kSampleLanes && kHist2Bins == kSampleLanes, "four counters to a lane, then one");
    fine[tid] = 0u;
    if (tid < 6) edge[tid] = 0u;
    __syncthreads();
    // A quarter of the samples, by their top digit: between which buckets the rest is worth counting.  Of four neighbours a different one
    // each time: where a layout's period is a multiple of four, the first ones are a biased quarter.  Twenty standard deviations of
    // independent samples' ranks, because these are no more independent than the rest: too few cost a window without an end, too many
    // only a coarser digit.
    constexpr uint32_t kFew = kSamples / 4;
#pragma unroll
    for (int j = 0; j < kSampleLoads; ++j) count_digit(h, true, key[4 * j + (j & 3)] >> kKeyShift, true, lane, 1u);
    __syncthreads();
    // counts before a lane's `sum`
    auto before = [&](uint32_t sum, uint32_t* tmp) __attribute__((always_inline)) {
        const uint32_t incl = wave_scan_incl(sum);
        if (lane == 63) tmp[wave] = incl;
        __syncthreads();
        const uint32_t one = lane < NW ? tmp[lane] : 0u, upto = wave_scan_incl(one);
        return (uint32_t)__builtin_amdgcn_readlane((int)(upto - one), wave) + incl - sum;
    };
    auto clamped = [](float r, uint32_t most) __attribute__((always_inline)) { return r < 1.f ? 1u : (r > (float)most ? most : (uint32_t)r); };
    const float share = (float)k / (float)L;
    {
        const uint4 v = reinterpret_cast<const uint4*>(h)[kHistBins / 4 - 1 - tid];
        const uint32_t cnt[4] = {v.w, v.z, v.y, v.x};  // from the top down
        uint32_t run = before(v.x + v.y + v.z + v.w, sums[0]);
        const float at = share * kFew, wide = 20.f * sqrtf(share * (1.f - share) * kFew) + 20.f;
        const uint32_t r0 = clamped(at - wide, kFew), r1 = clamped(at + wide, kFew), r2 = clamped(at, kFew);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t b = (uint32_t)(kHistBins - 1 - 4 * tid - i), end = run + cnt[i];
            if (run < r0 && end >= r0) {
                edge[0] = b;
                edge[3] = run;
            }
            if (run < r1 && end >= r1) {
                edge[1] = b;
                edge[4] = end;
            }
            if (run < r2 && end >= r2) edge[2] = b;
            run = end;
        }
        __syncthreads();
    }
    const uint32_t top = edge[0], bottom = edge[1], middle = edge[2] << kKeyShift;  // top >= bottom
    const bool crowded = edge[4] - edge[3] > kFew / 2;                              // many of them may be the same
    // All that lie between, by 2^10 digits of what there is between; how many are above; the differences.
    const uint32_t base = bottom << kKeyShift, range = ((top - bottom + 1u) << kKeyShift) - 1u;
    const int shift = 32 - __clz((int)range) - kHist2Bits;  // at least 9
    uint32_t above = 0, off = 0;
#pragma unroll
    for (int j = 0; j < kSampleLoads; ++j) {
        int in = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t x = key[4 * j + i], d = x - base;
            above += x > base + range ? 1u : 0u;
            in += x >= middle ? 1 : 0;
            if (crowded)
                count_digit(fine, d <= range, d >> shift, true, lane, 1u);
            else if (d <= range)
                atomicAdd(&fine[d >> shift], 1u);
        }
        in += __builtin_amdgcn_mov_dpp(in, 0xB1, 0xF, 0xF, false);  // of the lanes of a stretch
        if constexpr (SHARE > 1) in += __builtin_amdgcn_mov_dpp(in, 0x4E, 0xF, 0xF, false);
        const int next = __builtin_amdgcn_update_dpp(in, in, 0x100 + (1 << SHARE), 0xF, 0xF, false);  // a stretch on; itself in a row's last one
        off += (uint32_t)((next - in) * (next - in));
    }
    above = wave_sum(above);
    off = wave_sum(off);
    if (lane == 0) {
        sums[1][wave] = above;
        sums[2][wave] = off;
    }
    __syncthreads();
    above = wave_sum(lane < NW ? sums[1][lane] : 0u);
    off = wave_sum(lane < NW ? sums[2][lane] : 0u);
    // half of the differences, each seen by all lanes of a stretch, and one fewer to a row of sixteen lanes than it has stretches
    constexpr float kRow = 16 >> SHARE, kSeen = 0.5f / (1 << SHARE) * (kRow / (kRow - 1.f));
    const float wide = kSampleDeviations * sqrtf(sample_variance((float)off * kSeen, k, L, present)) + sample_margin(L, present);
    const float at = share * kSamples;
    const uint32_t r0 = clamped(at - wide, kSamples), r1 = clamped(at + wide, kSamples), digit = (uint32_t)(kHist2Bins - 1 - tid);
    const uint32_t cnt = fine[digit], run = above + before(cnt, sums[0]), end = run + cnt;
    // where a rank lies outside what was counted there is no bound on that side; a zero is never a candidate
    auto atleast1 = [](uint32_t lo) __attribute__((always_inline)) { return lo ? lo : 1u; };
    if (tid == 0) {
        if (at - wide < 1.f || above >= r0) sel[c * 8 + 1] = 0x7FFFFFFFu;
        if (at + wide > (float)kSamples) sel[c * 8] = 1u;
    }
    if (at - wide >= 1.f && run < r0 && end >= r0) {
        const uint32_t hi = base + (digit << shift) + ((1u << shift) - 1u);
        sel[c * 8 + 1] = hi < 0x7FFFFFFFu ? hi : 0x7FFFFFFFu;
    }
    if (at + wide <= (float)kSamples) {
        if (run < r1 && end >= r1) sel[c * 8] = atleast1(base + (digit << shift));
        if (tid == kSampleLanes - 1 && end < r1) sel[c * 8] = 1u;
    }
    // (above < r0 <= end of the last digit, unless fewer are counted than r0)
    if (tid == kSampleLanes - 1 && end < r0) sel[c * 8 + 1] = 0x7FFFFFFFu;
    if (tid == 0 && above >= r1 && at + wide <= (float)kSamples) sel[c * 8] = atleast1(base);
}

// --------------------------------------------------------------- collect ----
// Per tile: count and range of the bins kept outright, and the candidates in bin order.
//
// Bound by the read of the spectrum.  Binary32 bins pass through LDS: a wave's own rows are half of every line of their
// run, and fetching each line for two waves was slower (62 M samples in chunks of 2^20: 52 against 44 us).  Samples
// lie in order, and binary16 bins are half the bytes: those are read straight into registers, without the barrier
// (62 M samples 51 -> 42, binary16 32 -> 29).
// A tile of more than kListCap candidates that are all the same value (the zeros past the end of a gradient, say) is marked,
// so that k_resolve can take it as one.
// FIND: every workgroup finds the threshold's bucket itself, from hist, instead of a launch before this one.  That is 16 KB more to
// read per tile, from cache, so it is done where the launch weighs more: see find_in_collect.
// WINDOW: sel holds the two keys between which candidates lie (k_sample) instead of the bucket; a candidate is its key, which is a sample's
// component too.
// clear (FIND only): the records, whose code words this kernel then clears, for a k_emit that finds the threshold itself.
template <bool FIND, bool TABLE, bool REAL, bool HALF, bool WINDOW = false>
__global__ __launch_bounds__(NT) void k_collect(const typename Stored<REAL, HALF>::T* __restrict__ spec, Shape u,
                                                const uint32_t* __restrict__ hist, uint32_t* __restrict__ sel,
                                                uint32_t* __restrict__ tinfo, uint32_t* __restrict__ tscan,
                                                uint2* __restrict__ cand, uint8_t* __restrict__ clear, TableArg<TABLE> tab, size_t n)
{
    using E = typename Elem<REAL>::T;
    __shared__ uint32_t wcnt[4], wdef[4], wvmax[4];
    __shared__ uint2 wsame[4];  // the one candidate value of a wave, or kMixed
    constexpr uint32_t kMixed = 0xFFFFFFFFu;  // no key
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Place at = place_of_tile<TABLE>(u, tab);
    const uint32_t B = at.B, tbase = at.tile * kTile, row0 = (uint32_t)wave * WAVE_BINS;
    const int pair_log = at.pair_log;
    const typename Stored<REAL, HALF>::T* X = spec + at.spec + tbase;
    const uint32_t count = units_in_tile<REAL>(n, at.chunk, B, tbase);
    uint32_t bstar = 0, lowest = 0, highest = 0;
    if constexpr (WINDOW) {
        lowest = sel[(size_t)at.chunk * 8];
        highest = sel[(size_t)at.chunk * 8 + 1];
    } else if constexpr (!FIND) {
        bstar = sel[(size_t)at.chunk * 8];
    }
    E z[ROWS];
    if constexpr (REAL || HALF) {
        load_units(X, row0, count, lane, pair_log, z);
    } else {
        __shared__ __align__(16) E stage[kTile];
        tile_to_lds(X, count, TABLE || (u.sstride & 1u) == 0, stage, tid);
        __syncthreads();
        load_units(stage, row0, count, lane, pair_log, z);
    }
    if constexpr (FIND) {
        if (clear) {  // the tile's share of the record behind the bitmap
            uint32_t* codes = reinterpret_cast<uint32_t*>(clear + at.record) + 4 + at.W;
            const uint32_t words = (uint32_t)(at.S / 4) - 4u - at.W, share = (words + at.Tn - 1u) / at.Tn;
            const uint32_t from = at.tile * share, to = from + share < words ? from + share : words;
            for (uint32_t i = from + (uint32_t)tid; i < to; i += NT) codes[i] = 0u;
        }
    }
    if constexpr (FIND) {
        const Bucket b = find_bucket(hist + (size_t)at.chunk * kHistBins, at.k);
        bstar = b.star;
        if (at.tile == 0 && tid == 0) *reinterpret_cast<uint2*>(sel + (size_t)at.chunk * 8) = make_uint2(b.star, b.need);
    }
    uint32_t key[ROWS], vb[ROWS];
    uint64_t cm[ROWS];
    uint32_t ndef = 0, vmax = 0, ncand = 0, mine = 0;  // mine: bit r set = this lane's bin of row r is a candidate
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const bool valid = tbase + row0 + (uint32_t)(r * 64 + lane) < B;
        key[r] = key_of(z[r]);
        vb[r] = vbits_of(z[r]);
        const uint32_t bucket = key[r] >> kKeyShift;
        const bool isdef = valid && (WINDOW ? key[r] > highest : bucket > bstar);
        const bool iscand = valid && (WINDOW ? key[r] - lowest <= highest - lowest : bucket == bstar);
        if (isdef) {
            ++ndef;
            vmax = vb[r] > vmax ? vb[r] : vmax;
        }
        mine |= (uint32_t)iscand << r;
        cm[r] = __ballot(iscand);
        ncand += (uint32_t)__popcll(cm[r]);
    }
    ndef = wave_sum(ndef);
    vmax = wave_max(vmax);
    uint2 same = make_uint2(kMixed, 0u);
    if (ncand > kListCap / 4) {
        uint32_t most_key = 0, most_vb = 0, least_key = 0, least_vb = 0;  // least: of the complements
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const bool in = (mine >> r) & 1u;
            most_key = in && key[r] > most_key ? key[r] : most_key;
            most_vb = in && vb[r] > most_vb ? vb[r] : most_vb;
            least_key = in && ~key[r] > least_key ? ~key[r] : least_key;
            least_vb = in && ~vb[r] > least_vb ? ~vb[r] : least_vb;
        }
        most_key = wave_max(most_key);
        most_vb = wave_max(most_vb);
        if (most_key == ~wave_max(least_key) && most_vb == ~wave_max(least_vb)) same = make_uint2(most_key, most_vb);
    }
    if (lane == 0) {
        wsame[wave] = same;
        wcnt[wave] = ncand;
        wdef[wave] = ndef;
        wvmax[wave] = vmax;
    }
    __syncthreads();
    uint32_t off = 0;
    for (int w = 0; w < wave; ++w) off += wcnt[w];
    uint2* out = cand + blockIdx.x * (size_t)kTile;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        if ((mine >> r) & 1u) {
            if constexpr (WINDOW)
                reinterpret_cast<uint32_t*>(cand)[blockIdx.x * (size_t)kTile + off + prefix_popc(cm[r])] = key[r];
            else
                out[off + prefix_popc(cm[r])] = make_uint2(key[r], vb[r]);
        }
        off += (uint32_t)__popcll(cm[r]);
    }
    if (tid == 64 && at.Tn > kFewTiles)  // counters of k_count_digit
        *reinterpret_cast<uint2*>(tscan + (size_t)blockIdx.x * 2) = make_uint2(0u, 0u);
    if (tid == 0) {
        uint32_t* ti = tinfo + (size_t)blockIdx.x * 4;
        ti[0] = wdef[0] + wdef[1] + wdef[2] + wdef[3];
        uint32_t m = wvmax[0];
        m = wvmax[1] > m ? wvmax[1] : m;
        m = wvmax[2] > m ? wvmax[2] : m;
        m = wvmax[3] > m ? wvmax[3] : m;
        ti[1] = m;
        const uint32_t all = wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3];
        uint2 one = make_uint2(kMixed, 0u);
        bool alike = all > kListCap;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint2 v = wsame[w];
            if (one.x == kMixed && wcnt[w]) one = v;
            alike = alike && (wcnt[w] == 0 || (v.x != kMixed && v.x == one.x && v.y == one.y));
        }
        ti[2] = all;
        ti[3] = alike ? 1u : 0u;
    }
}

// --------------------------------------------------------------- resolve ----
constexpr int RT = 1024;           // lanes of the per-chunk workgroups of the decoder's prefix kernels
constexpr int RW = RT / 64;        // 16 waves
constexpr int MAX_TILES = ((1 << (kMaxLogL - 1)) + 1 + kTile - 1) / kTile;  // 1025

// Launches with chunks of more than kKeptTiles tiles: what k_resolve would do in its two sweeps over the candidates is done before it by
// a workgroup per kPartTiles tiles, because a single one is bound by what a compute unit issues (a chunk of 2^22: 35 us).
// k_count_digit counts the candidates' second digit into the first kHist2Bins words of the chunk's tscan, which k_collect
// has cleared.  k_mark adds the candidates above the two digits' common prefix to their tiles' counts and maxima and moves
// the ones that share it to the front of their tile's list, unless they are more than k_resolve lists.
// Senders in us, without / with: one chunk of 2^22 90 / 70, thirty-three 801 / 785.  Chunks of 512 and 513 tiles no longer come
// here, since k_resolve holds as many candidates in registers: with / held there, chunks of 2^21 one 50.8 / 48.4, eight 119 / 115,
// thirty-two 355 / 351; Top-k chunks of 2^20 one 37.0 / 31.0, eight 59.2 / 49.6, thirty-two 117 / 109, sixty 193 / 182.
// Beside longer chunks, for which the two kernels run anyway, they do better here too: senders of tensors of 2^21 and 2^22 held / here 91.5 /
// 83.6, of six and one 142 / 132.
constexpr uint32_t kPartTiles = 64, kPartWave = kPartTiles / (NT / 64);
inline uint32_t parts_of(uint32_t tiles) { return (tiles + kPartTiles - 1u) / kPartTiles; }
static_assert(2 * (kFewTiles + 1) <= (uint32_t)kHist2Bins && 2 * 512 >= kHist2Bins, "a chunk of 512 tiles, the next length, holds the counters");
template <bool TABLE>
__device__ __forceinline__ Place part_of(const Shape& u, const TableArg<TABLE>& tab, const LongStarts& at, uint32_t& first)
{
    if constexpr (TABLE) {
        const LongShare share = long_share(at);
        first = share.blk * kPartTiles;
        return place_of<TABLE>(u, tab, share.tensor, 0u);
    } else {
        const uint32_t parts = (u.Tn + kPartTiles - 1u) / kPartTiles;
        first = blockIdx.x % parts * kPartTiles;
        return place_of<TABLE>(u, tab, blockIdx.x / parts, 0u);
    }
}
// The candidates of a wave's tiles [t0, t0 + kPartWave): tile(t, info, e) with a lane's candidate of the first row of 64.
template <typename Tile>
__device__ __forceinline__ void tiles_of_part(const uint4* ti, const uint2* cd, uint32_t t0, uint32_t Tn, int lane,
                                              Tile&& tile)
{
    constexpr int AHEAD = 8;
    static_assert(kPartWave % AHEAD == 0, "whole batches");
    for (uint32_t b = t0; b < t0 + kPartWave && b < Tn; b += AHEAD) {
        uint2 e[AHEAD];
#pragma unroll
        for (int v = 0; v < AHEAD; ++v)  // slots behind a tile's last candidate are allocated; what they hold is dropped
            e[v] = cd[(size_t)(b + v < Tn ? b + v : b) * kTile + lane];
#pragma unroll
        for (int v = 0; v < AHEAD; ++v)
            if (b + v < Tn) tile(b + v, ti[b + v], e[v]);
    }
}
template <bool TABLE>
__global__ __launch_bounds__(NT) void k_count_digit(Shape u, const uint32_t* __restrict__ tinfo, uint32_t* __restrict__ tscan,
                                                    const uint2* __restrict__ cand, TableArg<TABLE> tab, LongStarts at)
{
    __shared__ uint32_t h[kHist2Bins];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t first;
    const Place p = part_of<TABLE>(u, tab, at, first);
    for (int i = tid; i < kHist2Bins; i += NT) h[i] = 0u;
    __syncthreads();
    const uint2* cd = cand + p.tile0 * (size_t)kTile;
    tiles_of_part(reinterpret_cast<const uint4*>(tinfo) + p.tile0, cd, first + (uint32_t)wave * kPartWave, p.Tn, lane,
                  [&](uint32_t t, uint4 info, uint2 e) __attribute__((always_inline)) {
                      const uint32_t nc = info.w ? (info.z ? 1u : 0u) : info.z, weight = info.w ? info.z : 1u;
                      for (uint32_t i0 = 0; i0 < nc; i0 += 64u) {
                          const bool valid = i0 + (uint32_t)lane < nc;
                          if (i0) e = cd[(size_t)t * kTile + (valid ? i0 + (uint32_t)lane : 0u)];
                          count_digit(h, valid, (e.x >> kHist2Shift) & (uint32_t)(kHist2Bins - 1), i0 != 0, lane, weight);
                      }
                  });
    __syncthreads();
    uint32_t* g = tscan + (size_t)p.tile0 * 2;
    for (int i = tid; i < kHist2Bins; i += NT)
        if (h[i]) atomicAdd(&g[i], h[i]);
}
// the second digit of the threshold's key from its counts, by a whole workgroup of LANES lanes; need as k_find_bucket's
template <int LANES>
__device__ __forceinline__ void second_digit(const uint32_t* h, uint32_t need, uint32_t* tmp, uint32_t& s_digit, uint32_t& s_need,
                                             uint32_t& s_count)
{
    constexpr int PER = kHist2Bins / LANES;
    static_assert(PER >= 1, "a lane scans whole counters");
    // scan from the top digit down
    uint32_t cnt[PER], sum = 0;
    const int base = kHist2Bins - PER - (int)threadIdx.x * PER;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        cnt[i] = h[base + i];
        sum += cnt[i];
    }
    uint32_t run = block_scan_incl<LANES / 64>(sum, tmp) - sum;
#pragma unroll
    for (int i = PER - 1; i >= 0; --i) {
        if (run < need && run + cnt[i] >= need) {
            s_digit = (uint32_t)(base + i);
            s_need = need - run;
            s_count = cnt[i];
        }
        run += cnt[i];
    }
    __syncthreads();
}
template <bool TABLE>
__global__ __launch_bounds__(NT) void k_mark(Shape u, const uint32_t* __restrict__ sel, uint32_t* __restrict__ tinfo,
                                             const uint32_t* __restrict__ tscan, uint2* __restrict__ cand, TableArg<TABLE> tab,
                                             LongStarts at)
{
    __shared__ uint32_t tmp[NT / 64], s_digit, s_need, s_count;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t first;
    const Place p = part_of<TABLE>(u, tab, at, first);
    const uint32_t bstar = sel[p.chunk * 8 + 0], need = sel[p.chunk * 8 + 1];
    if (tid == 0) s_digit = s_need = s_count = 0u;
    second_digit<NT>(tscan + (size_t)p.tile0 * 2, need, tmp, s_digit, s_need, s_count);
    if (need == 0 || s_count > kListCap) return;
    const int prefix = (int)((bstar << kHist2Bits) | s_digit);
    uint4* ti = reinterpret_cast<uint4*>(tinfo) + p.tile0;
    uint2* cd = cand + p.tile0 * (size_t)kTile;
    const uint32_t t0 = first + (uint32_t)wave * kPartWave;
    uint32_t vm = 0;
    tiles_of_part(ti, cd, t0, p.Tn, lane, [&](uint32_t t, uint4 info, uint2 e) __attribute__((always_inline)) {
        const uint32_t nc = info.w ? (info.z ? 1u : 0u) : info.z, weight = info.w ? info.z : 1u;
        uint32_t more = 0, same = 0;
        for (uint32_t i0 = 0; i0 < nc; i0 += 64u) {
            const bool valid = i0 + (uint32_t)lane < nc;
            if (i0) e = cd[(size_t)t * kTile + (valid ? i0 + (uint32_t)lane : 0u)];
            const int top = valid ? (int)(e.x >> kHist2Shift) : -1;
            more += (uint32_t)__popcll(__ballot(top > prefix)) * weight;
            vm = top > prefix && e.y > vm ? e.y : vm;
            // a tile taken as one has more than kListCap candidates, so its digit is not this one
            const uint64_t m = __ballot(top == prefix);
            if (top == prefix) cd[(size_t)t * kTile + same + prefix_popc(m)] = e;  // never past the row it comes from
            same += (uint32_t)__popcll(m);
        }
        if (lane == 0) ti[t] = make_uint4(info.x + more, info.y, same, 0u);
    });
    vm = wave_max(vm);
    if (lane == 0 && vm && t0 < p.Tn) {
        uint32_t* y = &tinfo[((size_t)p.tile0 + t0) * 4 + 1];  // the maximum is the chunk's: any tile will do
        *y = vm > *y ? vm : *y;
    }
}

// One workgroup per chunk: finish the radix select on the candidates, break ties by bin order, scan the tiles, find the
// survivors' largest component, write the record header and zero the code words that two tiles will share.
//
// Bound by latency: of memory once, then of LDS and of the barriers, since a wave has a few instructions for each of its
// tiles.  So the candidates and the tiles' summaries are asked for together, before anything else, and stay in registers: a wave
// holds its tiles' first rows of 64 candidates (a tile has about 40) and its lanes their summaries.  The first sweep counts the
// candidates' second digit.  The second one counts per tile those above the two digits' common prefix, takes their range and
// lists the few that share it (ten or so of a million bins).  The list settles the threshold, and its members are added to
// their tiles afterwards.  More than kListCap of them (runs of equal keys) take a third digit and a third sweep.  Scans
// over counters and tiles are short, so every wave does them for itself instead of waiting at a barrier.  What happens rarely
// (more than 64 candidates in a tile, more than two listed by one lane) is kept out of the sweeps' straight code: jumping over it
// there cost a fetch from memory per tile, about 550 cycles.
// Measured, us per launch, against sweeps over LDS: one chunk of 2^16 6.2 -> 5.0, four of 2^18 9.3 -> 6.1, eight of 2^19 13.3 -> 7.2, four
// of 2^20 14.8 -> 11.4, sixty 18.3 -> 14.1.
// A tile whose candidates are all the same value is one candidate of its weight: 10^6 samples in chunks of 2^18, the last
// one nearly empty, Top-k sender and receiver 661 -> 72 us.
// Counting the second digit in k_collect instead saved a sweep here but cost that kernel more (43 -> 52 us: its atomics
// meet in memory).
//
// MERGED: every workgroup of k_emit does this for its own tile, which saves the launch; see resolve_in_emit.  The code words are
// clear already, and the tile of number 0 writes the headers.
// FETCH: tiles of a wave asked for at once; it holds twice as many.
constexpr int kFetch = 9, kFetchMost = 17;
template <int NW, int FETCH>
constexpr uint32_t kHeldTiles = 2 * FETCH * NW;
static_assert(kHeldTiles<16, kFetchMost> >= kKeptTiles && kHeldTiles<16, kFetch> == kFewTiles && kHeldTiles<NT / 64, kFetch> >= kMergedTiles,
              "the candidates stay in registers");
template <int MOST>
struct ResolveScratch {
    uint32_t h[kHist2Bins], list[kListCap], list_at[kListCap], list_vb[kListCap];
    uint32_t tgt[MOST], teq[MOST], take[MOST];
    uint2 sums[RW];  // of a wave's tiles: bins above the candidates, and candidates
    uint32_t listed, vmax;
};
struct ResolveArgs {
    int bits, m;
    uint32_t static_vmax, codes_per_bin;
};
struct Threshold {
    uint32_t tau, quota, pbase;  // quota: bins equal to tau that are kept, or ~0: all of them
    uint32_t rank0, eq0;         // MERGED: survivors, and bins equal to tau, before the tile
};
// A digit's counters, so that the sixteen a lane scans are read without bank conflicts.
__device__ __forceinline__ uint32_t digit_place(uint32_t d) { return ((d & 15u) << 6) | (d >> 4); }
static_assert(kHist2Bins == 1024, "sixteen counters to a lane");
struct Digit {
    uint32_t digit, need, count;  // all zero if no digit qualifies
};
// The digit of the need-th largest from its counters, by a single wave.
__device__ __forceinline__ Digit find_digit(const uint32_t* h, uint32_t need, int lane)
{
    uint32_t cnt[16], sum = 0;
    const int l = 63 - lane;  // from the top down
#pragma unroll
    for (int i = 0; i < 16; ++i) cnt[i] = h[i * 64 + l];
#pragma unroll
    for (int i = 0; i < 16; ++i) sum += cnt[i];
    uint32_t run = wave_scan_incl(sum) - sum;
    const uint64_t mine = __ballot(run < need && run + sum >= need);
    if (!mine) return Digit{0u, 0u, 0u};
    Digit d{0u, 0u, 0u};
#pragma unroll
    for (int i = 15; i >= 0; --i) {
        if (run < need && run + cnt[i] >= need) d = Digit{(uint32_t)(l * 16 + i), need - run, cnt[i]};
        run += cnt[i];
    }
    const int who = __ffsll((unsigned long long)mine) - 1;
    return Digit{(uint32_t)__builtin_amdgcn_readlane((int)d.digit, who), (uint32_t)__builtin_amdgcn_readlane((int)d.need, who),
                 (uint32_t)__builtin_amdgcn_readlane((int)d.count, who)};
}

// The threshold of a chunk of samples from the samples themselves, where the candidates do not have it: ten bits at a time, then every tile's
// samples above it and equal to it.  All but never needed (see k_sample), and slow, one workgroup reading the chunk five times: a sender of 62 M samples whose
// sample misleads in one of sixty chunks of 2^20, or in all of them, takes 900 to 1080 us instead of 135, one of 20 M in chunks of 2^18 330 instead of 59.
template <int LANES>
__device__ __forceinline__ Digit select_samples(const float* __restrict__ X, uint32_t present, uint32_t L, uint32_t Tn, uint32_t need,
                                                          uint32_t* h, uint32_t* tgt, uint32_t* teq, uint32_t& vm)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int AHEAD = 4;
    static_assert((1 << 18) % (4 * AHEAD * LANES) == 0 && kTile % (4 * AHEAD * 64) == 0, "whole batches");
    // keys i .. i + 3 of the chunk, with nothing but zeros past the gradient's end
    auto four = [&](uint32_t i) __attribute__((always_inline)) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i + 4u <= present) {
            v = *reinterpret_cast<const float4*>(X + i);
        } else if (i < present) {
            v.x = X[i];
            if (i + 1u < present) v.y = X[i + 1u];
            if (i + 2u < present) v.z = X[i + 2u];
        }
        return make_uint4(key_of(v.x), key_of(v.y), key_of(v.z), key_of(v.w));
    };
    Digit found{0u, need, 0u};
    uint32_t tau = 0;
    for (int top = 31; top > 0;) {
        const int shift = top > 10 ? top - 10 : 0;
        __syncthreads();
        for (int i = tid; i < kHist2Bins; i += LANES) h[i] = 0u;
        __syncthreads();
#pragma unroll 1
        for (uint32_t i = 0; i < L; i += 4 * AHEAD * LANES) {
            uint4 v[AHEAD];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) v[q] = four(i + 4u * (uint32_t)(q * LANES + tid));
            auto count = [&](uint32_t key) __attribute__((always_inline)) {
                count_digit(h, key >> top == tau, digit_place((key >> shift) & ((1u << (top - shift)) - 1u)), true, lane, 1u);
            };
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) {
                count(v[q].x);
                count(v[q].y);
                count(v[q].z);
                count(v[q].w);
            }
        }
        __syncthreads();
        found = find_digit(h, found.need, lane);
        tau = tau << (top - shift) | found.digit;
        top = shift;
    }
    __syncthreads();
    uint32_t most = 0;
    for (uint32_t t = (uint32_t)wave; t < Tn; t += LANES / 64) {
        uint32_t above = 0, same = 0;
#pragma unroll 1
        for (uint32_t i = 0; i < (uint32_t)kTile; i += 4 * AHEAD * 64) {
            uint4 v[AHEAD];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) v[q] = four(t * kTile + i + 4u * (uint32_t)(q * 64 + lane));
            auto count = [&](uint32_t key) __attribute__((always_inline)) {
                above += (uint32_t)__popcll(__ballot(key > tau));
                same += (uint32_t)__popcll(__ballot(key == tau));
                most = key > most ? key : most;
            };
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) {
                count(v[q].x);
                count(v[q].y);
                count(v[q].z);
                count(v[q].w);
            }
        }
        if (lane == 0) {
            tgt[t] = above;
            teq[t] = same;
        }
    }
    vm = most;  // the largest sample is a survivor
    __syncthreads();
    return Digit{tau, found.need, found.count};
}

// WINDOW: samples (time domain); the candidates lie between two keys, and X has them all, `present` of them in the chunk.
template <int NW, int FETCH, bool MERGED, bool WINDOW, int MOST>
__device__ __forceinline__ Threshold resolve_chunk(const Place& at, const ResolveArgs& a, ResolveScratch<MOST>& lds,
                                                   uint32_t* __restrict__ sel, const uint32_t* __restrict__ tinfo,
                                                   uint32_t* __restrict__ tscan, const uint2* __restrict__ cand,
                                                   uint8_t* __restrict__ records, uint8_t* __restrict__ stream, const HeaderInfo& hdr,
                                                   const float* __restrict__ X, uint32_t present)
{
    constexpr int LANES = NW * 64, HELD = 2 * FETCH;
    uint32_t *const h = lds.h, *const list = lds.list, *const list_at = lds.list_at, *const list_vb = lds.list_vb;
    uint32_t *const tgt = lds.tgt, *const teq = lds.teq;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t c = at.chunk;
    const uint32_t Tn = at.Tn, k = at.k, W = at.W;
    const uint4* ti = reinterpret_cast<const uint4*>(tinfo + (size_t)at.tile0 * 4);
    const uint2* cd = cand + at.tile0 * (size_t)kTile;
    // WINDOW: the lowest candidate's key and the highest one's; a key's digits are those of what it lies above the lowest
    const uint32_t bstar = sel[c * 8 + 0];
    uint32_t need = sel[c * 8 + 1];
    const uint32_t lowest = WINDOW ? bstar : 0u, range = WINDOW ? need - bstar : 0u;
    const int low = WINDOW ? (range >> kHist2Bits ? 32 - __clz((int)range) - kHist2Bits : 0) : kHist2Shift;  // bits below the first digit
    auto rel = [&](uint32_t key) __attribute__((always_inline)) { return WINDOW ? key - lowest : key; };
    const bool counted = !MERGED && !WINDOW && Tn > kHeldTiles<NW, FETCH>;  // k_count_digit and k_mark have been here

    // A wave's tiles are wave, wave + NW, ...; lane v has the summary of the v-th, e[v] its first candidates: of a sample the key is all there
    // is, and a lane has two of them.  Slots behind a tile's last candidate are allocated; what they hold is dropped.
    constexpr uint32_t ROW = WINDOW ? 128u : 64u;
    const uint32_t* ck = reinterpret_cast<const uint32_t*>(cand) + at.tile0 * (size_t)kTile;
    auto first_of = [&](uint32_t t) __attribute__((always_inline)) {
        return WINDOW ? *reinterpret_cast<const uint2*>(ck + (size_t)t * kTile + 2 * lane) : cd[(size_t)t * kTile + lane];
    };
    auto one_of = [&](uint32_t t, uint32_t i) __attribute__((always_inline)) {
        return WINDOW ? make_uint2(ck[(size_t)t * kTile + i], ck[(size_t)t * kTile + i]) : cd[(size_t)t * kTile + i];
    };
    const uint32_t own = (uint32_t)wave + (uint32_t)(lane * NW);
    const bool holds = !counted && lane < HELD && own < Tn, second = !counted && (uint32_t)(wave + FETCH * NW) < Tn;
    uint4 info = make_uint4(0u, 0u, 0u, 0u);
    uint2 e[HELD];
#pragma unroll
    for (int v = 0; v < HELD; ++v) e[v] = make_uint2(0u, 0u);
    if (holds) info = ti[own];
    if (!counted && !WINDOW) {
#pragma unroll
        for (int v = 0; v < FETCH; ++v) {
            const uint32_t t = (uint32_t)(wave + v * NW);
            e[v] = first_of(t < Tn ? t : 0u);
        }
    }
    if (second && !WINDOW) {
#pragma unroll
        for (int v = FETCH; v < HELD; ++v) {
            const uint32_t t = (uint32_t)(wave + v * NW);
            e[v] = first_of(t < Tn ? t : 0u);
        }
    }
    for (int i = tid; i < kHist2Bins; i += LANES) h[i] = 0u;
    if (tid == 0) lds.listed = lds.vmax = 0u;
    uint32_t vm = info.y;  // per-lane maximum over survivors
    if (holds) {
        tgt[own] = info.x;
        teq[own] = 0u;
    }
    if (counted)
        for (uint32_t t = tid; t < Tn; t += LANES) {
            const uint4 v = ti[t];
            tgt[t] = v.x;
            teq[t] = 0u;
            lds.take[t] = v.z;  // what k_mark has left
            vm = v.y > vm ? v.y : vm;
        }
    if constexpr (WINDOW) {
        const uint32_t defs = wave_sum(info.x), cands = wave_sum(info.z);
        if (lane == 0) lds.sums[wave] = make_uint2(defs, cands);
    }
    __syncthreads();
    bool missed = false, zero = false;  // the threshold is not among the candidates; it is zero
    bool unkept = false;                // all that is kept are candidates
    if constexpr (WINDOW) {
        const uint2 v = lane < NW ? lds.sums[lane] : make_uint2(0u, 0u);
        const uint32_t defs = wave_sum(v.x), cands = wave_sum(v.y);
        need = k - defs;
        missed = k != 0 && (defs >= k || need > cands);
        zero = missed && defs < k && lowest == 1u;
        unkept = defs == 0u;
        if (zero) need -= cands;
    }
    const bool any = need > 0 || missed;  // else nothing is kept (k = 0), and there are no candidates
    // candidates of the lane's tile to look at, each standing for `weight` of them
    const uint32_t ncand = info.w ? (info.z ? 1u : 0u) : info.z, nweight = info.w ? info.z : 1u;
    const bool heavy = __any(ncand > ROW);

    // f(v, nc, weight) for the first row of candidates of each of this wave's tiles: straight code, and as little of it as
    // can be, because it runs once and is fetched as it runs
    auto first_rows = [&](auto&& f) __attribute__((always_inline)) {
        auto one = [&](int v, uint2 x) __attribute__((always_inline)) {
            f(v, x, (uint32_t)__builtin_amdgcn_readlane((int)ncand, v), (uint32_t)__builtin_amdgcn_readlane((int)nweight, v));
        };
        if constexpr (WINDOW) {
            // a loop, with the next tiles' rows on their way, that goes through memory both times: it takes as long as rows held in registers,
            // and a fourth of the code
            constexpr int AHEAD = 4;
            uint2 a[AHEAD], b[AHEAD];
            auto ask = [&](uint2 (&x)[AHEAD], int v) __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < AHEAD; ++q) {
                    const uint32_t t = (uint32_t)(wave + (v + q) * NW);
                    x[q] = first_of(t < Tn ? t : 0u);
                }
            };
            ask(a, 0);
#pragma unroll 1
            for (int v = 0; (uint32_t)(wave + v * NW) < Tn; v += 2 * AHEAD) {
                ask(b, v + AHEAD);
#pragma unroll
                for (int q = 0; q < AHEAD; ++q) one(v + q, a[q]);
                ask(a, v + 2 * AHEAD);
#pragma unroll
                for (int q = 0; q < AHEAD; ++q) one(v + AHEAD + q, b[q]);
            }
        } else {
#pragma unroll
            for (int v = 0; v < HELD; ++v) {
                if (v == FETCH && !second) break;
                one(v, e[v]);
            }
        }
    };
    static_assert(HELD + 8 <= 64, "a lane to every tile that is asked for");
    // row(t, i0, e, valid, weight) for all rows of the wave's tiles from number `from` on, out of memory
    auto rows_of_memory = [&](uint32_t from, auto&& row) __attribute__((always_inline)) {
        for (uint32_t t = (uint32_t)wave; t < Tn; t += NW) {
            const uint4 v = ti[t];
            const uint32_t nc = v.w ? (v.z ? 1u : 0u) : v.z;
            for (uint32_t i0 = from; i0 < nc; i0 += 64u) {
                const bool valid = i0 + (uint32_t)lane < nc;
                row(t, i0, one_of(t, valid ? i0 + (uint32_t)lane : 0u), valid, v.w ? v.z : 1u);
            }
        }
    };
    // row(t, i0, e, valid, weight) for the rows behind the first of those of the wave's tiles that have any (a tile taken as one has none);
    // of samples several tiles' second rows asked for at a time
    auto more_rows = [&](auto&& row) __attribute__((always_inline)) {
        if constexpr (!WINDOW) {
            rows_of_memory(ROW, row);
            return;
        }
        constexpr int AHEAD = 8;
        for (uint64_t left = __ballot(ncand > ROW); left;) {
            uint2 x[AHEAD];
            uint32_t tiles[AHEAD], counts[AHEAD];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) {
                const int v = left ? __ffsll((unsigned long long)left) - 1 : 0;
                tiles[q] = (uint32_t)(wave + v * NW);
                counts[q] = left ? (uint32_t)__builtin_amdgcn_readlane((int)ncand, v) : 0u;
                x[q] = one_of(tiles[q], ROW + (uint32_t)lane);
                left &= left - 1u;
            }
#pragma unroll
            for (int q = 0; q < AHEAD; ++q)
                if (counts[q]) row(tiles[q], ROW, x[q], ROW + (uint32_t)lane < counts[q], 1u);
#pragma unroll 1
            for (int q = 0; q < AHEAD; ++q)
                for (uint32_t i0 = ROW + 64u; i0 < counts[q]; i0 += 64u) {
                    const bool valid = i0 + (uint32_t)lane < counts[q];
                    row(tiles[q], i0, one_of(tiles[q], valid ? i0 + (uint32_t)lane : 0u), valid, 1u);
                }
        }
    };
    // row(t, key, valid, weight) for all rows of samples
    auto every_row = [&](auto&& row) __attribute__((always_inline)) {
        first_rows([&](int v, uint2 x, uint32_t nc, uint32_t weight) __attribute__((always_inline)) {
            row((uint32_t)(wave + v * NW), x.x, 2u * (uint32_t)lane < nc, weight);
            row((uint32_t)(wave + v * NW), x.y, 2u * (uint32_t)lane + 1u < nc, weight);
        });
        if (heavy)
            more_rows([&](uint32_t t, uint32_t, uint2 x, bool valid, uint32_t weight) __attribute__((always_inline)) { row(t, x.x, valid, weight); });
    };
    auto digit_of = [&](uint32_t key) __attribute__((always_inline)) {
        return digit_place((rel(key) >> low) & (uint32_t)(kHist2Bins - 1));
    };
    if (missed) {
    } else if (any && counted) {
        for (int i = tid; i < kHist2Bins; i += LANES) h[digit_place((uint32_t)i)] = tscan[(size_t)at.tile0 * 2 + i];
    } else if (any) {
        first_rows([&](int v, uint2 x, uint32_t nc, uint32_t weight) __attribute__((always_inline)) {
            if constexpr (WINDOW) {
                if (2u * (uint32_t)lane < nc) atomicAdd(&h[digit_of(x.x)], weight);
                if (2u * (uint32_t)lane + 1u < nc) atomicAdd(&h[digit_of(x.y)], weight);
            } else {
                if ((uint32_t)lane < nc) atomicAdd(&h[digit_of(x.x)], weight);
            }
        });
        if (heavy)
            more_rows([&](uint32_t, uint32_t, uint2 x, bool valid, uint32_t weight) __attribute__((always_inline)) {
                count_digit(h, valid, digit_of(x.x), true, lane, weight);
            });
    }
    __syncthreads();
    Digit found = any && !missed ? find_digit(h, need, lane) : Digit{0u, need, 0u};
    need = found.need;
    uint32_t equal = found.count;
    const int prefix = (int)(WINDOW ? found.digit : (bstar << kHist2Bits) | found.digit);  // the top bits of the threshold's key
    const bool few = equal <= kListCap && !missed;
    uint32_t tau = any ? (uint32_t)prefix << low : 0xFFFFFFFFu, quota = 0;  // WINDOW: above the lowest, until it is known
    bool ties = false;
    if (WINDOW && zero) {  // all that are not zero are kept, and the first zeros
        if (holds) {
            tgt[own] += info.z;
            teq[own] = (uint32_t)kTile - info.x - info.z;
        }
        if (unkept)
            every_row([&](uint32_t, uint32_t x, bool valid, uint32_t) __attribute__((always_inline)) { vm = valid && x > vm ? x : vm; });
        tau = 0u;
        quota = need;
        ties = true;  // a quota of all of them is one, too
        __syncthreads();
    } else if (WINDOW && missed) {
        const Digit d = select_samples<LANES>(X, present, Tn * (uint32_t)kTile, Tn, k, h, tgt, teq, vm);
        tau = d.digit;
        quota = d.need;
        equal = d.count;
        ties = equal != quota;
    } else if (any && few) {
        auto list_one = [&](uint32_t place, uint2 x) __attribute__((always_inline)) {
            const uint32_t slot = atomicAdd(&lds.listed, 1u);
            if (slot < kListCap) {
                list[slot] = rel(x.x);
                list_at[slot] = place;
                list_vb[slot] = x.y;
            }
        };
        if (counted) {
            for (uint32_t t = tid; t < Tn; t += LANES)
                for (uint32_t i = 0, n = lds.take[t]; i < n; ++i) list_one(t * (uint32_t)kTile + i, cd[(size_t)t * kTile + i]);
        } else {
            // a tile taken as one has more than kListCap candidates, so its digit is not the one with few
            uint32_t above = 0, hits = 0;  // lane v: of the wave's v-th tile; each lane: what it has to list, the last two of it
            uint32_t hit_at[2] = {0u, 0u};
            uint2 hit[2] = {make_uint2(0u, 0u), make_uint2(0u, 0u)};
            first_rows([&](int v, uint2 x, uint32_t nc, uint32_t weight) __attribute__((always_inline)) {
                auto hit_one = [&](bool is, uint32_t place, uint32_t key, uint32_t vb) __attribute__((always_inline)) {
                    hits += is ? 1u : 0u;
                    hit_at[1] = is ? hit_at[0] : hit_at[1];
                    hit[1].x = is ? hit[0].x : hit[1].x;
                    hit[1].y = is ? hit[0].y : hit[1].y;
                    hit_at[0] = is ? place : hit_at[0];
                    hit[0].x = is ? key : hit[0].x;
                    hit[0].y = is ? vb : hit[0].y;
                };
                if constexpr (WINDOW) {
                    const int top = 2u * (uint32_t)lane < nc ? (int)(rel(x.x) >> low) : -1;
                    const int next = 2u * (uint32_t)lane + 1u < nc ? (int)(rel(x.y) >> low) : -1;
                    const uint32_t many = (uint32_t)(__popcll(__ballot(top > prefix)) + __popcll(__ballot(next > prefix))) * weight;
                    above = lane == v ? many : above;
                    vm = top > prefix && x.x > vm ? x.x : vm;
                    vm = next > prefix && x.y > vm ? x.y : vm;
                    const uint32_t place = (uint32_t)(wave + v * NW) * (uint32_t)kTile + 2u * (uint32_t)lane;
                    if (top == prefix) list_one(place, make_uint2(x.x, x.x));
                    if (next == prefix) list_one(place + 1u, make_uint2(x.y, x.y));
                } else {
                    const int top = (uint32_t)lane < nc ? (int)(rel(x.x) >> low) : -1;
                    const uint32_t many = (uint32_t)__popcll(__ballot(top > prefix)) * weight;
                    above = lane == v ? many : above;
                    vm = top > prefix && x.y > vm ? x.y : vm;
                    hit_one(top == prefix, (uint32_t)v, x.x, x.y);
                }
            });
            if (holds) atomicAdd(&tgt[own], above);
            if (WINDOW) {
            } else if (!__any(hits > 2u)) {
#pragma unroll
                for (uint32_t i = 0; i < 2u; ++i)
                    if (hits > i) list_one(((uint32_t)wave + hit_at[i] * NW) * (uint32_t)kTile + (uint32_t)lane, hit[i]);
            } else {
                rows_of_memory(0u, [&](uint32_t t, uint32_t i0, uint2 x, bool valid, uint32_t) __attribute__((always_inline)) {
                    if (i0 == 0u && valid && (int)(x.x >> low) == prefix) list_one(t * (uint32_t)kTile + (uint32_t)lane, x);
                });
            }
            if (heavy)
                more_rows([&](uint32_t t, uint32_t i0, uint2 x, bool valid, uint32_t weight) __attribute__((always_inline)) {
                    const int top = valid ? (int)(rel(x.x) >> low) : -1;
                    const uint64_t more = __ballot(top > prefix);
                    vm = top > prefix && x.y > vm ? x.y : vm;
                    if (more && lane == 0) atomicAdd(&tgt[t], (uint32_t)__popcll(more) * weight);
                    if (top == prefix) list_one(t * (uint32_t)kTile + i0 + (uint32_t)lane, x);
                });
        }
        __syncthreads();
        const uint32_t listed = equal;
        search_list<4>(list, listed, low, lane, tau, need, equal);
        quota = need;
        ties = equal != quota;
        for (uint32_t i = tid; i < listed; i += LANES) {
            const uint32_t x = list[i], place = list_at[i];
            bool kept = x >= tau;
            if (ties && x == tau) {  // the first of them, in bin order
                uint32_t before = 0;
                for (uint32_t j = 0; j < listed; ++j) before += list[j] == tau && list_at[j] < place;
                kept = before < quota;
                atomicAdd(&teq[place / (uint32_t)kTile], 1u);
            }
            if (kept) {
                atomicAdd(&tgt[place / (uint32_t)kTile], 1u);
                vm = list_vb[i] > vm ? list_vb[i] : vm;
            }
        }
        if constexpr (WINDOW) tau += lowest;
        __syncthreads();
    } else if (any) {
        if constexpr (WINDOW) {
            // Crowds are most often one value: a gradient on a grid, of 8 bits once.  Then it is known, and otherwise its bits are found, ten at a time.
            uint32_t least = 0, most = 0;  // least: of the complements
            every_row([&](uint32_t, uint32_t x, bool valid, uint32_t) __attribute__((always_inline)) {
                const bool in = valid && (int)(rel(x) >> low) == prefix;
                most = in && rel(x) > most ? rel(x) : most;
                least = in && ~rel(x) > least ? ~rel(x) : least;
            });
            least = wave_max(least);
            most = wave_max(most);
            if (lane == 0) lds.sums[wave] = make_uint2(least, most);
            __syncthreads();
            const uint2 v = lane < NW ? lds.sums[lane] : make_uint2(0u, 0u);
            most = wave_max(v.y);
            const bool one = most == ~wave_max(v.x);
            if (one) tau = most;
            for (int top = one ? 0 : low; top > 0;) {
                const int shift = top > kHist2Bits ? top - kHist2Bits : 0;
                __syncthreads();
                for (int i = tid; i < kHist2Bins; i += LANES) h[i] = 0u;
                __syncthreads();
                every_row([&](uint32_t, uint32_t x, bool valid, uint32_t weight) __attribute__((always_inline)) {
                    count_digit(h, valid && rel(x) >> top == tau >> top, digit_place((rel(x) >> shift) & ((1u << (top - shift)) - 1u)), true, lane, weight);
                });
                __syncthreads();
                found = find_digit(h, need, lane);
                tau |= found.digit << shift;
                need = found.need;
                equal = found.count;
                top = shift;
            }
        } else {
            __syncthreads();
            for (int i = tid; i < kHist2Bins; i += LANES) h[i] = 0u;
            __syncthreads();
            rows_of_memory(0u, [&](uint32_t, uint32_t, uint2 x, bool valid, uint32_t weight) __attribute__((always_inline)) {
                count_digit(h, valid && (int)(x.x >> kHist2Shift) == prefix, digit_place(x.x & 511u), true, lane, weight);
            });
            __syncthreads();
            found = find_digit(h, need, lane);
            tau |= found.digit;
            need = found.need;
            equal = found.count;
        }
        quota = need;
        ties = equal != quota;
        if constexpr (WINDOW) tau += lowest;
        auto weigh = [&](uint32_t t, uint2 x, bool valid, uint32_t weight) __attribute__((always_inline)) {
            const uint64_t gm = __ballot(valid && x.x > tau), em = __ballot(valid && x.x == tau);
            if (gm && lane == 0) atomicAdd(&tgt[t], (uint32_t)__popcll(gm) * weight);
            if (em && lane == 0) atomicAdd(&teq[t], (uint32_t)__popcll(em) * weight);
            vm = valid && (ties ? x.x > tau : x.x >= tau) && x.y > vm ? x.y : vm;
        };
        if constexpr (WINDOW)
            every_row([&](uint32_t t, uint32_t x, bool valid, uint32_t weight) __attribute__((always_inline)) { weigh(t, make_uint2(x, x), valid, weight); });
        else
            rows_of_memory(0u, [&](uint32_t t, uint32_t, uint2 x, bool valid, uint32_t weight) __attribute__((always_inline)) { weigh(t, x, valid, weight); });
        __syncthreads();
    }
    const bool count_equal = any && !few;  // tgt does not hold the kept ones of the bins equal to tau yet

    // Scan over tiles: the equal keys before a tile decide who gets the tie quota, the survivors before it give the ranks.  Every
    // wave runs through all of them, 64 at a time, and sees to its share.
    uint32_t* rec = reinterpret_cast<uint32_t*>(records + at.record);
    uint32_t* codes = rec + 4 + W;
    const uint32_t twoN = a.codes_per_bin * (uint32_t)a.bits;  // code bits per kept bin
    uint32_t eqcarry = 0, rankcarry = 0, my_rank = 0, my_eq = 0;
    for (uint32_t t0 = 0; t0 < Tn; t0 += 64u) {
        const uint32_t t = t0 + (uint32_t)lane;
        const bool share = (t0 >> 6) % NW == (uint32_t)wave;
        uint32_t surv = t < Tn ? tgt[t] : 0u, eqpre = 0;
        if (ties || count_equal) {
            uint32_t eq = t < Tn ? teq[t] : 0u;
            if (ties) {
                const uint32_t incl = wave_scan_incl(eq);
                eqpre = eqcarry + incl - eq;
                eq = eqpre >= quota ? 0u : (eq < quota - eqpre ? eq : quota - eqpre);
                eqcarry += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            }
            if (count_equal) {
                surv += eq;
                if (share && t < Tn) lds.take[t] = eq;
            }
        }
        const uint32_t incl = wave_scan_incl(surv), before = rankcarry + incl - surv;
        rankcarry += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        // ranks never leave [0, k]: whatever the counts say, the code words of a tile stay inside the record
        const uint32_t rank = before < k ? before : k;
        if constexpr (MERGED) {
            if (at.tile >> 6 == t0 >> 6) {
                my_rank = (uint32_t)__builtin_amdgcn_readlane((int)rank, (int)(at.tile & 63u));
                my_eq = (uint32_t)__builtin_amdgcn_readlane((int)eqpre, (int)(at.tile & 63u));
            }
        } else if (share && t < Tn) {
            // where all bins equal to tau are taken, a prefix of zero (and an endless quota) says so
            *reinterpret_cast<uint2*>(tscan + (size_t)(at.tile0 + t) * 2) = make_uint2(rank, eqpre);
            surv = surv < k - rank ? surv : k - rank;
            if (surv) {
                codes[(twoN * rank) >> 5] = 0u;
                codes[(twoN * (rank + surv) - 1u) >> 5] = 0u;
            }
        }
    }
    if constexpr (!MERGED) {
        const uint32_t code_words = (twoN * k + 31u) >> 5, rec_words = (uint32_t)(at.S / 4) - 4u - W;
        for (uint32_t w = code_words + tid; w < rec_words; w += LANES) codes[w] = 0u;
    }

    // largest component over the survivors (not needed when the caller fixed the range: Sec. 3.2.1, static max)
    uint32_t vmax = a.static_vmax;
    if (!vmax) {
        if (count_equal && ties && !missed) {
            __syncthreads();
            for (uint32_t t = (uint32_t)wave; t < Tn; t += NW) {
                const uint4 v = ti[t];
                const uint32_t nc = v.w ? (v.z ? 1u : 0u) : v.z, take = lds.take[t];
                uint32_t eqseen = 0;  // bins of the tile equal to tau seen so far
                for (uint32_t i0 = 0; i0 < nc && eqseen < take; i0 += 64u) {
                    const bool valid = i0 + (uint32_t)lane < nc;
                    const uint2 x = one_of(t, valid ? i0 + (uint32_t)lane : 0u);
                    const bool iseq = valid && x.x == tau;
                    const uint64_t em = __ballot(iseq);
                    vm = iseq && eqseen + prefix_popc(em) < take && x.y > vm ? x.y : vm;
                    eqseen += (uint32_t)__popcll(em);
                }
            }
        }
        vm = wave_max(vm);
        if (lane == 0 && vm) atomicMax(&lds.vmax, vm);
        __syncthreads();
        vmax = lds.vmax;
    }
    Threshold th{tau, ties ? quota : 0xFFFFFFFFu, 0u, 0u, 0u};
    if (a.bits != 32) {
        const int64_t pb = (int64_t)(vmax >> (23 - a.m)) - (int64_t)((1u << (a.bits - 1)) - 2u);
        th.pbase = pb < 1 ? 1u : (uint32_t)pb;
    }
    if constexpr (MERGED) {
        th.rank0 = my_rank;
        th.eq0 = my_eq;
    } else if (tid == 0) {
        sel[c * 8 + 2] = th.tau;
        sel[c * 8 + 3] = th.quota;
        sel[c * 8 + 4] = th.pbase;
        sel[c * 8 + 5] = vmax;
    }
    if ((!MERGED || at.tile == 0) && tid == 0) *reinterpret_cast<uint4*>(rec) = make_uint4(th.pbase, vmax, k, at.word3);
    if (hdr.write && c == 0 && (!MERGED || at.tile == 0) && tid < 16) reinterpret_cast<uint32_t*>(stream)[tid] = header_word(hdr, tid);
    return th;
}
template <bool TABLE, bool WINDOW, int NW, int FETCH>
__global__ __launch_bounds__(NW * 64) void k_resolve(Shape u, ResolveArgs a, uint32_t* __restrict__ sel, const uint32_t* __restrict__ tinfo,
                                                     uint32_t* __restrict__ tscan, const uint2* __restrict__ cand,
                                                     uint8_t* __restrict__ records, uint8_t* __restrict__ stream,
                                                     HeaderInfo hdr, TableArg<TABLE> tab, const float* __restrict__ samples, size_t n)
{
    __shared__ ResolveScratch<MAX_TILES> lds;
    const Place at = place_of<TABLE>(u, tab, blockIdx.x, 0u);
    resolve_chunk<NW, FETCH, false, WINDOW>(at, a, lds, sel, tinfo, tscan, cand, records, stream, hdr, WINDOW ? samples + at.spec : nullptr,
                                            WINDOW ? present_of<true>(n, at.chunk, at.B) : 0u);
}

// ------------------------------------------------------------------ emit ----
// Per tile: flags, ranks, Algorithm 1 codes, bit-packing, bitmap words.
//
// Bound by the latency of its loads and by instruction issue.  Everything about a row of 64 units that is the same for all its lanes (place in
// the tile, existing lanes, flags as a 64-bit mask, counts) is scalar, and bins
// come straight from memory into registers: by way of LDS, binary32 ones took as long, binary16 ones 50 us for 45.  Samples
// do pass through LDS, in 16-byte loads (50 us for 55).
// Measured, 62 M samples in chunks of 2^20, half of the bins kept as 8-bit codes, against shuffles and vector masks: 70 -> 67 us,
// binary16 bins 60 -> 45, 15 % of the samples kept at 32 bits 98 -> 50; one chunk of 2^16 8 -> 7.
// The last tiles come first: k_collect has just read them, and of what does not fit the 256 MB cache the first ones are gone
// (62 M samples in chunks of 2^20 67 -> 61 us, the step 537 -> 532; 138 M in 2^22 150 -> 138, 1320 -> 1306; top-k 223 -> 218.5).  After a kernel that
// wrote the bins instead of reading them the order makes no difference.  Eight by eight, so that a tile stays on the XCD whose L2 may have it from
// k_collect: one by one, calls of 100 to 450 tiles of 2^14 points lost 3 to 12 us.  Below kEmitBackwards tiles of 16 KB the first ones are still there, and
// the order stays.  Above it, forwards / backwards: senders 2^16 17 M 101.6 / 98.8, 60 M 303.0 / 295.2, 2^20 20 M 122.8 / 122.2, 62 M 322.4 / 315.7, 2^22 138 M 776 / 760, binary16 34 M
// 149.8 / 149.7; top-k 34 M 141.9 / 143.8, 62 M 244.5 / 237.5; tensors 18 of 2^20 195.3 / 193.7, 48 442.0 / 440.9, random sets of 60 298.8 / 299.9, 90 326.0 / 328.3, 150 460.4 / 461.0
// (builds differ by as much below the line, where the order is the same).
constexpr uint32_t kEmitBackwards = 4096;
// tiles from the first on whose order is reversed, a multiple of eight; an argument, since asking for the launch's size cost every launch 0.5 us
inline uint32_t emit_reversed(uint32_t tiles) { return tiles >= kEmitBackwards ? tiles & ~7u : 0u; }
template <bool TABLE, bool REAL, bool HALF, bool MERGED>
__global__ __launch_bounds__(NT) void k_emit(const typename Stored<REAL, HALF>::T* __restrict__ spec, Shape u, uint32_t reversed, ResolveArgs a,
                                             uint32_t* __restrict__ sel, uint32_t* __restrict__ tscan,
                                             const uint32_t* __restrict__ tinfo, const uint2* __restrict__ cand,
                                             uint8_t* __restrict__ records, uint8_t* __restrict__ stream, HeaderInfo hdr,
                                             TableArg<TABLE> tab, size_t n)
{
    using E = typename Elem<REAL>::T;
    constexpr uint32_t CODES = Elem<REAL>::kCodes;
    constexpr int CW = kTile * (int)CODES / 2 + 8;                       // words for codes of up to 16 bits, see shw
    __shared__ __align__(16) uint32_t cw[CW];
    __shared__ __align__(16) uint64_t bmw[kTile / 64];
    __shared__ uint32_t weq[4], wfl[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t nth = !MERGED && blockIdx.x < reversed ? reversed - 8u - (blockIdx.x & ~7u) + (blockIdx.x & 7u) : blockIdx.x;  // which tile of the launch
    const Place at = place_of_tile<TABLE>(u, tab, nth);
    const uint32_t c = at.chunk, tile = at.tile, B = at.B, W = at.W;
    const size_t S = at.S;
    const int pair_log = at.pair_log;
    const int bits = a.bits, m = a.m;
    Threshold found;
    if constexpr (!MERGED)
        found = Threshold{sel[c * 8 + 2], sel[c * 8 + 3], sel[c * 8 + 4], tscan[(size_t)nth * 2 + 0],
                          tscan[(size_t)nth * 2 + 1]};
    const uint32_t twoN = CODES * (uint32_t)bits;  // code bits per kept unit
    const int shift = 23 - m;

    const uint32_t tbase = tile * kTile, row0 = (uint32_t)wave * WAVE_BINS;  // row0: this wave's first unit in the tile
    const typename Stored<REAL, HALF>::T* X = spec + at.spec + tbase;
    const uint32_t count = units_in_tile<REAL>(n, c, B, tbase);
    E z[ROWS];
    if constexpr (REAL) {
        __shared__ __align__(16) E stage[kTile];
        tile_to_lds(X, count, true, stage, tid);  // chunks start on multiples of 32 samples of a 16-byte aligned gradient
        __syncthreads();
        load_units(stage, row0, count, lane, 0, z);
    } else {
        load_units(X, row0, count, lane, pair_log, z);
    }
    if constexpr (MERGED) {
        __shared__ ResolveScratch<kMergedTiles> lds;
        found = resolve_chunk<NT / 64, kFetch, true, false>(at, a, lds, sel, tinfo, tscan, cand, records, stream, hdr, nullptr, 0u);
    }
    const uint32_t tau = found.tau, quota = found.quota, pbase = found.pbase, rank0 = found.rank0, eq0 = found.eq0;
    if (bits != 32)  // 32-bit codes go straight to memory
        for (uint32_t i = 4u * tid; i < (uint32_t)kTile * twoN / 32u + 8u; i += 4u * NT)
            *reinterpret_cast<uint4*>(cw + i) = make_uint4(0u, 0u, 0u, 0u);
    uint64_t fm[ROWS];
    uint32_t nfl = 0;
    if (quota == 0xFFFFFFFFu) {  // every unit equal to the threshold is wanted
#pragma unroll
        for (int r = 0; r < ROWS; ++r) fm[r] = __ballot(key_of(z[r]) >= tau);
        if (tbase + (uint32_t)kTile > B) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) fm[r] &= row_mask(tbase + row0 + r * 64u, B);
        }
    } else {
        uint32_t key[ROWS], neq = 0;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            key[r] = key_of(z[r]);
            fm[r] = __ballot(key[r] == tau) & row_mask(tbase + row0 + r * 64u, B);
            neq += (uint32_t)__popcll(fm[r]);
        }
        if (lane == 0) weq[wave] = neq;
        __syncthreads();
        uint32_t eqrun = eq0;
#pragma unroll
        for (int w = 0; w < 3; ++w) eqrun += w < wave ? weq[w] : 0u;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint64_t em = fm[r];
            const bool eq = __builtin_amdgcn_inverse_ballot_w64(em);
            fm[r] = (__ballot(key[r] > tau) & row_mask(tbase + row0 + r * 64u, B)) | __ballot(eq && eqrun + prefix_popc(em) < quota);
            eqrun += (uint32_t)__popcll(em);
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) nfl += (uint32_t)__popcll(fm[r]);
    if (lane == 0) {
        wfl[wave] = nfl;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) bmw[wave * ROWS + r] = fm[r];
    }
    __syncthreads();
    uint32_t* rec = reinterpret_cast<uint32_t*>(records + at.record);
    uint32_t* bitmap = rec + 4;
    uint32_t* codes = bitmap + W;
    if (tid < kTile / 32) {
        const uint32_t wi = tile * (kTile / 32) + tid;
        if (wi < W) bitmap[wi] = reinterpret_cast<const uint32_t*>(bmw)[tid];
    }
    uint32_t rank = 0, total = 0;  // survivors of the tile before this wave's, and all of them
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)wfl[w]);
        rank += w < wave ? v : 0u;
        total += v;
    }
    if (total == 0) return;
    const uint32_t w0 = (twoN * rank0) >> 5;
    // The tile's code words are built in LDS at cw[shw + i] for the record's word w0 + i, with shw chosen so that an
    // LDS word and its place in memory are aligned alike: whole 16-byte groups then go out as one store each.
    const uint32_t shw = (uint32_t)((reinterpret_cast<uintptr_t>(codes + w0) >> 2) & 3u);
    // the one or two binary32 patterns a unit is coded from
    auto code = [&](const E& v, int h, int width) __attribute__((always_inline)) {
        if constexpr (REAL)
            return quantize(__float_as_uint(v), pbase, width, shift);
        else
            return quantize(__float_as_uint(h ? v.y : v.x), pbase, width, shift);
    };
    // put(unit, its rank inside the tile) for every survivor
    auto survivors = [&](auto&& put) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if (__builtin_amdgcn_inverse_ballot_w64(fm[r])) put(z[r], rank + prefix_popc(fm[r]));
            rank += (uint32_t)__popcll(fm[r]);
        }
    };
    if (bits == 32) {
        uint32_t* dst = codes + CODES * rank0;
        const uint32_t room = (uint32_t)(S / 4) - 4u - W;
        survivors([&](const E& v, uint32_t rk) {
            if (CODES * (rank0 + rk + 1u) > room) return;  // never, unless the counts of the tiles disagree
            if constexpr (REAL)
                dst[rk] = code(v, 0, 32);
            else
                store_code_pair(dst + 2u * rk, code(v, 0, 32), code(v, 1, 32));
        });
        return;
    }
    if (bits == 8) {
        // 8-bit codes: a survivor is one aligned 16-bit store (bin) or one byte (sample), no read-modify-write
        if constexpr (REAL) {
            uint8_t* dst = reinterpret_cast<uint8_t*>(cw) + (rank0 - 4u * w0 + 4u * shw);
            survivors([&](const E& v, uint32_t rk) { dst[rk] = (uint8_t)code(v, 0, 8); });
        } else {
            uint16_t* dst = reinterpret_cast<uint16_t*>(cw) + (rank0 - 2u * w0 + 2u * shw);
            survivors([&](const E& v, uint32_t rk) { dst[rk] = (uint16_t)(code(v, 0, 8) | (code(v, 1, 8) << 8)); });
        }
    } else {
        const uint32_t p0 = twoN * rank0 - (w0 << 5) + (shw << 5);  // first survivor's bit position inside cw
        survivors([&](const E& v, uint32_t rk) {
            uint32_t both = code(v, 0, bits);
            if constexpr (!REAL) both |= code(v, 1, bits) << bits;  // at most 32 bits
            const uint32_t p = p0 + twoN * rk, wi = p >> 5, sh = p & 31u;
            atomicOr(&cw[wi], both << sh);
            if (sh + twoN > 32u) atomicOr(&cw[wi + 1], both >> (32u - sh));
        });
    }
    __syncthreads();
    const uint32_t w1 = (twoN * (rank0 + total) - 1u) >> 5;
    const uint32_t rec_words = (uint32_t)(S / 4) - 4u - W;  // code words the record has room for
    const uint32_t nw_all = w1 - w0 + 1u;
    const uint32_t nw = w0 >= rec_words ? 0u : (nw_all < rec_words - w0 ? nw_all : rec_words - w0);
    // group g = LDS words 4g .. 4g+3 = record words w0 - shw + 4g .. (16-byte aligned in memory)
    const uint32_t groups = (shw + nw + 3u) >> 2;
    uint32_t* gbase = codes + w0 - shw;
    for (uint32_t g = tid; g < groups; g += NT) {
        const uint32_t i0 = 4u * g;  // LDS index of the group's first word; its tile word index is i0 - shw
        if (i0 >= shw + 1u && i0 + 3u + 1u < shw + nw) {
            // all four words lie strictly inside the tile's run
            *reinterpret_cast<uint4*>(gbase + i0) = *reinterpret_cast<const uint4*>(cw + i0);
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 4u; ++j) {
                const uint32_t li = i0 + j;
                if (li < shw || li >= shw + nw) continue;
                const uint32_t i = li - shw, v = cw[li];
                if (i == 0 || i == nw - 1u)
                    atomicOr(&codes[w0 + i], v);  // may be shared with the neighbouring tile (zeroed by k_resolve)
                else
                    codes[w0 + i] = v;
            }
        }
    }
}

// ---------------------------------------------------------------- decode ----
constexpr int GROUP_WORDS = 16;  // one wave of the decode kernel covers 512 bins = 16 bitmap words

// Number of set bits before each group of 16 bitmap words of a record (the prefix sum of Sec. 3.2's status vector, kept at the
// granularity a wave needs), for the part-th kPrefixWords words; the words before them are counted again, a lane's own loads and
// then eight of them in flight.  The word that the Nyquist bin has to itself makes no part of its own: the one before takes it along.
// The last part checks the headers and leaves the verdict in *verdict.  A workgroup per record took, us: sixty of 2^20 bins (Top-k)
// 9.1 -> 6.7, ResNet-50's tensors 11.7 -> 7.7, eight peers' sixty of 2^19 15.6 -> 14.1 (16.1 with parts of one word).
// Receivers of five peers' single chunk of 2^21 samples 43.2 -> 36.4, of 2^22 57.0 -> 51.3 (37.4 and 52.2 with those before asked for one by one).
// Short records, of a quad to a lane at most, are many and bound by instructions: they do a quarter of it, and what they have no use for lies out of
// their way.  Receivers of six peers' 380 chunks of 2^16, 8 bits 142.8 -> 141.2, eight peers' 700, 284.4 -> 280.9.
constexpr int kPrefixQuads = 4;  // four words each: what a lane has in flight
constexpr uint32_t kPrefixWords = 4u * kPrefixQuads * RT;
__host__ __device__ constexpr uint32_t prefix_parts(uint32_t W) { return W < 2u ? 1u : (W + kPrefixWords - 2u) / kPrefixWords; }
__device__ __forceinline__ void group_prefix_part(const uint8_t* __restrict__ stream, const uint8_t* __restrict__ record,
                                                  bool first_of_stream, uint32_t W, uint32_t k, uint32_t word3,
                                                  const HeaderInfo& hdr, uint32_t part, uint32_t* __restrict__ gprefix,
                                                  uint32_t* __restrict__ verdict)
{
    __shared__ uint32_t own[kPrefixQuads * RW], earlier[RW];
    static_assert(kPrefixQuads * RW == 64, "a lane to each of a part's sums");
    static_assert(GROUP_WORDS == 16, "a group is four lanes");
    const uint32_t parts = prefix_parts(W);
    if (part >= parts) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t* bitmap = reinterpret_cast<const uint32_t*>(record) + 4;
    const uint4* quads = reinterpret_cast<const uint4*>(bitmap);  // records and bitmaps are 16-byte aligned
    const uint32_t whole = W / 4u, from = part * kPrefixQuads * RT;
    auto ones = [](uint4 v) __attribute__((always_inline)) { return (uint32_t)(__popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w)); };
    const bool last = part + 1u == parts, along = last && W > parts * kPrefixWords;
    uint32_t nyquist = 0, before = 0;
    if (__builtin_expect(along, 0)) nyquist = scalar_load(bitmap + (W - 1u));
    const bool more = whole >= from + RT;  // than a quad to a lane
    uint4 v[kPrefixQuads];
    auto load = [&](int i) __attribute__((always_inline)) {
        const uint32_t q = from + (uint32_t)(i * RT + tid);
        v[i] = quads[q < whole ? q : 0u];
    };
    load(0);
    if (more)
#pragma unroll
        for (int i = 1; i < kPrefixQuads; ++i) load(i);
    if (__builtin_expect(part != 0u, 0))
#pragma unroll 2
        for (uint32_t p = 0; p < part; ++p)
#pragma unroll
            for (uint32_t i = 0; i < kPrefixQuads; ++i) before += ones(quads[(p * kPrefixQuads + i) * RT + (uint32_t)tid]);
    uint32_t incl[kPrefixQuads], sum[kPrefixQuads];
    auto count = [&](int i) __attribute__((always_inline)) {
        const uint32_t q = from + (uint32_t)(i * RT + tid);
        sum[i] = q < whole ? ones(v[i]) : 0u;
        if (q == whole)
            for (uint32_t w = 4u * q; w < W; ++w) sum[i] += (uint32_t)__popc(bitmap[w]);
        incl[i] = wave_scan_incl(sum[i]);
    };
    count(0);
#pragma unroll
    for (int i = 1; i < kPrefixQuads; ++i) sum[i] = incl[i] = 0u;
    if (more)
#pragma unroll
        for (int i = 1; i < kPrefixQuads; ++i) count(i);
#pragma unroll
    for (int i = 0; i < kPrefixQuads; ++i)
        if (lane == 63) own[i * RW + wave] = incl[i];
    if (__builtin_expect(part != 0u, 0)) {
        before = wave_sum(before);
        if (lane == 63) earlier[wave] = before;
    }
    __syncthreads();
    // every wave scans the sums for itself: read one by one they were 64 LDS reads a wave
    uint32_t run = 0;
    if (__builtin_expect(part != 0u, 0)) run = wave_sum(lane < RW ? earlier[lane] : 0u);
    const uint32_t one = own[lane], upto = wave_scan_incl(one);
    auto store = [&](int i) __attribute__((always_inline)) {
        const uint32_t here = run + (uint32_t)__builtin_amdgcn_readlane((int)(upto - one), i * RW + wave) + incl[i] - sum[i];
        const uint32_t q = from + (uint32_t)(i * RT + tid);
        if ((q & 3u) == 0u && 4u * q < W) gprefix[q >> 2] = here;
    };
    store(0);
    if (more)
#pragma unroll
        for (int i = 1; i < kPrefixQuads; ++i) store(i);
    run += (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    if (last && tid == 0) {
        if (__builtin_expect(along, 0)) gprefix[(W - 1u) / GROUP_WORDS] = run;
        *verdict = record_verdict(record, stream, first_of_stream, run + (uint32_t)__popc(nyquist), k, word3, hdr);
    }
}

template <bool TABLE>
__global__ __launch_bounds__(RT) void k_group_prefix(const uint8_t* __restrict__ stream,
                                                     const uint8_t* __restrict__ records, Shape u, HeaderInfo hdr, uint32_t parts,
                                                     uint32_t* __restrict__ gprefix, uint32_t* __restrict__ verdicts,
                                                     uint32_t* __restrict__ ctl, StatusNote note, TableArg<TABLE> tab)
{
    if (ctl && blockIdx.x == 0) clear_control(ctl, note, threadIdx.x, RT);
    const uint32_t c = blockIdx.x / parts;
    const Place at = place_of<TABLE>(u, tab, c, 0u);
    group_prefix_part(stream, records + at.record, c == 0, at.W, at.k, at.word3, hdr, blockIdx.x % parts, gprefix + at.group0, verdicts + c);
}

// The same for several peers' streams.
__global__ __launch_bounds__(RT) void k_group_prefix_peers(PeerList streams, uint32_t C, size_t S, uint32_t W, uint32_t k,
                                                           HeaderInfo hdr, uint32_t parts, uint32_t* __restrict__ gprefix,
                                                           uint32_t* __restrict__ verdicts, uint32_t* __restrict__ ctl,
                                                           StatusNote note)
{
    if (blockIdx.x == 0) clear_control(ctl, note, threadIdx.x, RT);
    const uint32_t r = blockIdx.x / parts, peer = r / C, c = r % C;
    const uint32_t G = (W + GROUP_WORDS - 1) / GROUP_WORDS;
    const uint8_t* stream = streams.p[peer];
    group_prefix_part(stream, stream + 64 + (size_t)c * S, c == 0, W, k, 0u, hdr, blockIdx.x % parts, gprefix + (size_t)r * G, verdicts + r);
}

// What a wave needs of one record to decode its 512 units (16 bitmap words, group g of the chunk).
template <int NL>
struct WaveCodes {
    uint64_t fm[ROWS];   // kept units of each row
    uint32_t run;        // kept units of the chunk before the wave's
    uint32_t pbase;      // from the record's header
    uint32_t rel;        // bit position of the wave's first code inside its window
    u32x4 main[NL ? NL : 1], tail;
};

// NL: 16-byte loads per lane.  The codes of a wave's kept units are one contiguous byte range of the record.  Up to 16 bits
// wide they are fetched as a window of NL * 1024 + 16 bytes from the 16-byte boundary below the first one (lanes past the
// last code's 16 bytes repeat them), and picked out of LDS by rank; 32-bit codes (NL = 0) need no unpacking and are read by
// rank from memory, a row's being adjacent.  The header, the bitmap words and the prefix are scalar loads.
template <int NL>
__device__ __forceinline__ void fetch_flags(const uint8_t* __restrict__ record, uint32_t W, uint32_t g, int lane, WaveCodes<NL>& wc)
{
    const uint32_t* rec = reinterpret_cast<const uint32_t*>(record);
    const uint32_t w0 = g * GROUP_WORDS;
    wc.pbase = scalar_load(rec);
    if (w0 + GROUP_WORDS <= W) {
        const uint64_t* p = reinterpret_cast<const uint64_t*>(rec + 4 + w0);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) wc.fm[r] = scalar_load(p + r);
    } else {
        const uint32_t w = w0 + (uint32_t)lane, v = w < W ? rec[4 + w] : 0u;
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            wc.fm[r] = (uint32_t)__builtin_amdgcn_readlane((int)v, 2 * r) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)v, 2 * r + 1) << 32);
    }
}
// The codes of the wave's units; run, kept: kept units before them and among them (or an upper bound).
template <int NL, uint32_t CODES>
__device__ __forceinline__ void fetch_codes(const uint8_t* __restrict__ record, size_t S, uint32_t W, int bits, uint32_t run,
                                            uint32_t kept, int lane, WaveCodes<NL>& wc)
{
    wc.run = run;
    if constexpr (NL > 0) {
        const uint32_t width = CODES * (uint32_t)bits, last = (uint32_t)S - 16u;  // S is a multiple of 16, at least 32
        const uint32_t first = 8u * (16u + 4u * W) + width * wc.run;             // bit position in the record
        const uint32_t start = (first >> 3) & ~15u, end = (first + width * kept) >> 3 & ~15u;
        const uint32_t lim = end < last ? end : last;  // a corrupt bitmap must not point outside the record
        wc.rel = first - 8u * start;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const uint32_t off = start + (uint32_t)(i * 1024 + lane * 16);
            wc.main[i] = *reinterpret_cast<const u32x4*>(record + (off < lim ? off : lim));
        }
        const uint32_t off = start + (uint32_t)(NL * 1024);
        wc.tail = *reinterpret_cast<const u32x4*>(record + (off < lim ? off : lim));
    }
}

// Kept units before a wave's and among them (or an upper bound), from the chunk's group prefixes.
__device__ __forceinline__ void group_run(const uint32_t* __restrict__ gprefix, uint32_t W, uint32_t g, uint32_t& run, uint32_t& kept)
{
    const uint32_t w0 = g * GROUP_WORDS;
    run = scalar_load(gprefix + (w0 < W ? g : 0u));
    kept = w0 + GROUP_WORDS < W ? scalar_load(gprefix + g + 1u) - run : (uint32_t)WAVE_BINS;
}

template <int NL>
constexpr int kWindow = NL * 1024 + 32;  // bytes of LDS per wave: the window and slack for a two-word read
typedef u32x4 __attribute__((may_alias)) u32x4_any;
typedef uint32_t __attribute__((may_alias)) u32_any;
typedef uint16_t __attribute__((may_alias)) u16_any;

// put(row, value) for all rows, zero where a unit is not kept.  The window is the wave's own: no barrier.
template <int NL, bool REAL, typename Put>
__device__ __forceinline__ void unpack_codes(const WaveCodes<NL>& wc, const uint8_t* __restrict__ record, size_t S, uint32_t W,
                                             int bits, int shift, int lane, uint8_t* window, Put&& put)
{
    using E = typename Elem<REAL>::T;
    constexpr uint32_t CODES = Elem<REAL>::kCodes;
    if constexpr (NL == 0) {
        const uint32_t* codes = reinterpret_cast<const uint32_t*>(record) + 4 + W;
        const uint32_t room = (uint32_t)(S / 4) - 4u - W;  // code words the record has room for
        E v[ROWS];
        uint32_t first = CODES * wc.run;  // a row's first code
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint32_t at = first + CODES * prefix_popc(wc.fm[r]);
            v[r] = Elem<REAL>::zero();
            if (__builtin_amdgcn_inverse_ballot_w64(wc.fm[r]) && at + CODES <= room) __builtin_memcpy(&v[r], codes + at, sizeof(E));
            first += CODES * (uint32_t)__popcll(wc.fm[r]);
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) put(r, v[r]);
    } else {
#pragma unroll
        for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4_any*>(window + i * 1024 + lane * 16) = wc.main[i];
        if (lane == 0) *reinterpret_cast<u32x4_any*>(window + NL * 1024) = wc.tail;
        __builtin_amdgcn_wave_barrier();
        uint32_t base = (wc.pbase - 1u) << shift;
        asm("" : "+v"(base));  // in a vector register, so that it is the addend of a shift-and-add
        auto rows = [&](auto narrow) __attribute__((always_inline)) {
            constexpr bool BYTES = decltype(narrow)::value;
            const uint32_t nb = BYTES ? 8u : (uint32_t)bits;
            uint32_t raw[ROWS];
            uint32_t at = BYTES ? wc.rel >> 3 : wc.rel;  // a row's first code in the window, in bytes or bits
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const uint32_t rank = prefix_popc(wc.fm[r]), kept = (uint32_t)__popcll(wc.fm[r]);
                if constexpr (BYTES && REAL) {
                    raw[r] = window[at + rank];
                    at += kept;
                } else if constexpr (BYTES) {
                    raw[r] = *reinterpret_cast<const u16_any*>(window + (at + 2u * rank));
                    at += 2u * kept;
                } else {
                    const uint32_t p = at + CODES * nb * rank;
                    const u32_any* w = reinterpret_cast<const u32_any*>(window + 4u * (p >> 5));
                    raw[r] = __builtin_amdgcn_alignbit(w[1], w[0], p);  // a unit's codes are at most 32 bits
                    at += CODES * nb * kept;
                }
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const uint32_t codes = __builtin_amdgcn_inverse_ballot_w64(wc.fm[r]) ? raw[r] : 0u;
                if constexpr (REAL) {
                    put(r, __uint_as_float(dequantize_field(codes, 0u, nb, base, shift)));
                } else {
                    put(r, make_float2(__uint_as_float(dequantize_field(codes, 0u, nb, base, shift)),
                                       __uint_as_float(dequantize_field(codes, nb, nb, base, shift))));
                }
            }
        };
        if (NL == 1 && bits == 8)
            rows(std::true_type{});
        else
            rows(std::false_type{});
        __builtin_amdgcn_wave_barrier();
    }
}

// The wave's units to their slots of a staged tile (see load_units).
template <typename T>
__device__ __forceinline__ void place_units(T* stage, uint32_t row0, int lane, int pair_log, const T (&z)[ROWS])
{
    if (pair_log == 0) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) stage[row0 + (uint32_t)(lane + r * 64)] = z[r];
        return;
    }
    const uint32_t N1 = 1u << pair_log, half = N1 / 2;
    if (pair_log >= 10) {
        const uint32_t run = row0 & ~(N1 - 1u), k1 = row0 - run;
        if (k1 < half) {
            T* p = stage + run + 2u * (k1 + (uint32_t)lane);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) p[r * 128] = z[r];
        } else {
            const uint32_t last = run + 2u * (N1 - k1 - 64u * (ROWS - 1) - (uint32_t)lane) + 1u;  // row ROWS-1
            T* p = stage + last;
#pragma unroll
            for (int r = 1; r < ROWS; ++r) p[(ROWS - 1 - r) * 128] = z[r];
            stage[k1 == half && lane == 0 ? run + 1u : last + 128u * (ROWS - 1)] = z[0];
        }
    } else {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint32_t row = row0 + (uint32_t)r * 64u, run = row & ~(N1 - 1u), k1 = row - run;
            const uint32_t slot = k1 < half ? run + 2u * (k1 + (uint32_t)lane) : run + 2u * (N1 - k1 - (uint32_t)lane) + 1u;
            stage[k1 == half && lane == 0 ? run + 1u : slot] = z[r];
        }
    }
}

// A staged tile to memory.  vec: the spectrum buffer is the codec's own (chunks padded to 16 bins, 16-byte aligned):
// 16-byte stores, whose last one may reach past the chunk's last bin into the padding.
template <typename T>
__device__ __forceinline__ void tile_from_lds(T* __restrict__ X, const T* stage, uint32_t count, bool vec, int tid)
{
    constexpr int PER = 16 / (int)sizeof(T);
    if (vec) {
        float4* dst = reinterpret_cast<float4*>(X);
        const float4* src = reinterpret_cast<const float4*>(stage);
#pragma unroll
        for (int i = 0; i < kTile / PER / NT; ++i) {
            const uint32_t idx = (uint32_t)(tid + i * NT);
            if ((uint32_t)PER * idx < count) dst[idx] = src[idx];
        }
    } else {
        for (uint32_t i = tid; i < count; i += NT) X[i] = stage[i];
    }
}

// One stream: a workgroup per tile, a wave per 512 units.
// REAL: time-domain records (one code per kept sample); `spec` is then the gradient itself, chunk stride B = L
// samples, written up to sample n only.
// HALF: the spectrum is written as binary16 pairs (half-precision variant).
//
// Bound by the stores of the decoded units, and by instruction issue: everything that is the same for a row's 64 lanes
// (its flags as a mask, counts, addresses) is scalar.  Two dependent round trips (bitmap and prefix, then codes) are
// covered by the seven workgroups that a compute unit holds.
// COUNT: a workgroup counts the bits before its tile itself, leaves the record's verdict and the control block, and
// there is no launch before this one: see prefix_in_decode.
// Measured, 62 M samples in chunks of 2^20, against persistent workgroups with software-pipelined loads whose flags and
// ranks were per lane: half of the bins kept as 8-bit codes 62 -> 54 us (298 MB of traffic), binary16 bins 52 -> 33, 15 % of
// the samples kept at 32 bits 93 -> 62; chunks of 2^22 (138 M samples) 136 -> 112.
template <int NL, bool COUNT, bool TABLE, bool REAL, bool HALF>
__global__ __launch_bounds__(NT) void k_decode(const uint8_t* __restrict__ stream, const uint8_t* __restrict__ records, Shape u,
                                               int bits, int m, const uint32_t* __restrict__ gprefix, HeaderInfo hdr,
                                               uint32_t* __restrict__ verdicts, uint32_t* __restrict__ ctl, StatusNote note,
                                               typename Stored<REAL, HALF>::T* __restrict__ spec, bool vec,
                                               TableArg<TABLE> tab, size_t n)
{
    using T = typename Stored<REAL, HALF>::T;
    __shared__ __align__(16) uint8_t windows[NL ? 4 * kWindow<NL> : 16];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Place at = place_of_tile<TABLE>(u, tab);
    const uint32_t W = at.W, tbase = at.tile * kTile, row0 = (uint32_t)wave * WAVE_BINS;
    const size_t S = at.S;
    const uint8_t* record = records + at.record;
    uint8_t* window = windows + (NL ? wave * kWindow<NL> : 0);
    WaveCodes<NL> wc;
    const uint32_t g = at.tile * (kTile / 32 / GROUP_WORDS) + wave;  // this wave's group of bitmap words
    uint32_t run, kept;
    if constexpr (!COUNT) group_run(gprefix + at.group0, W, g, run, kept);
    fetch_flags<NL>(record, W, g, lane, wc);
    if constexpr (COUNT) {
        __shared__ uint32_t before[NT / 64], own[NT / 64];
        kept = 0;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) kept += (uint32_t)__popcll(wc.fm[r]);
        const uint4* words = reinterpret_cast<const uint4*>(record + 16);
        uint32_t mine = 0;  // set bits of the tiles before this one
        for (uint32_t i = (uint32_t)tid; i < at.tile * (kTile / 128u); i += NT) {
            const uint4 v = words[i];
            mine += (uint32_t)(__popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w));
        }
        mine = wave_sum(mine);
        if (lane == 0) {
            before[wave] = mine;
            own[wave] = kept;
        }
        __syncthreads();
        uint32_t total = 0;
        run = 0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) {
            total += before[w] + own[w];
            run += before[w] + (w < wave ? own[w] : 0u);
        }
        run = (uint32_t)__builtin_amdgcn_readfirstlane((int)run);
        if (at.tile + 1u == at.Tn && tid == 0)  // the last tile has seen all of the bitmap
            verdicts[at.chunk] = record_verdict(record, stream, at.chunk == 0, total, at.k, at.word3, hdr);
        if (ctl && blockIdx.x == 0) clear_control(ctl, note, tid, NT);
    }
    fetch_codes<NL, Elem<REAL>::kCodes>(record, S, W, bits, run, kept, lane, wc);
    T z[ROWS];
    unpack_codes<NL, REAL>(wc, record, S, W, bits, 23 - m, lane, window, [&](int r, const typename Elem<REAL>::T& v) {
        if constexpr (HALF)
            z[r] = pack_half2(v);
        else
            z[r] = v;
    });
    T* X = spec + at.spec + tbase;
    const uint32_t count = units_in_tile<REAL>(n, at.chunk, at.B, tbase);
    if constexpr (REAL) {
        X += row0 + (uint32_t)lane;
        if (count == (uint32_t)kTile) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) X[r * 64] = z[r];
        } else {
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
                if (row0 + (uint32_t)(r * 64 + lane) < count) X[r * 64] = z[r];
        }
    } else {
        __shared__ __align__(16) T stage[kTile];
        place_units(stage, row0, lane, at.pair_log, z);
        __syncthreads();
        tile_from_lds(X, stage, count, vec, tid);
    }
}

// Several peers' streams (receiver under an allgather: Sec. 4, implementation): the units summed over the peers in list order in
// registers, starting from zero, and stored once.
//
// Codes of up to 15 bits: a lane has eight neighbouring bins.  Their codes are neighbours in the record, so it fetches one window
// and shifts them out of registers (Stretch; ByteWindow for 8-bit codes): no LDS, and nothing scalar for each row of 64 bins.  While one peer's
// are unpacked the next one's window and the byte of the bitmap after that are on their way.
// Measured, eight peers of 62 M samples, half of the bins kept as 8-bit codes, against 64 neighbouring lanes a row and codes picked out
// of LDS by rank (k_decode_peers_wide, still there for the widest codes): 178 -> 155 us with Stretch, 131 with ByteWindow.
//
// What bounds it: with Stretch instruction issue (26 a bin and peer), with ByteWindow the trips to memory of 551 MB (106 us for a copy of
// as much), of which a wave has one window and one byte a lane of flags on the way.  What counts there is eight waves a SIMD: two windows ahead and
// seven waves took 136, three sets of registers in turn and four waves 178, workgroups that go on to another tile with its first
// window fetched before 203.
// A load of more than four bytes a lane, or of lanes that are not neighbours, takes the vector memory's return path 17 cycles; one whose lanes
// start inside a word 33 for eight bytes and 66 for sixteen.  Adds, logic of up to three operands, binary32 arithmetic and shifts by a
// constant hold a SIMD for two cycles, nearly everything else for four: permutes, bit-field and bit-select operations, shifts by a
// register, counts, minima, comparisons and selections by one.

// Eight neighbouring bins of a record of 8-bit codes: a kept bin is two bytes, so those of eight are in the four words from the first one's on, or,
// where it starts inside a word and all are kept, the first byte pair of the next lane's window too.  Two byte permutes deal the bytes of
// four bins out, by selectors looked up for the set of them that is kept.
// For three bits of mantissa a code with its sign in the top bit goes to its place by one arithmetic shift and a mask that drops the copies
// of the sign, and the base is added where the bin is kept, by a mask looked up with the selectors.  Kept bins with a zero code, which comparisons
// and selections would sort out one by one, are looked for in the four words first: waves that have one, 1 in 20 or so, and other codes take
// dequantize_field.
struct ByteTable {
    uint4 pick[16];  // entry i, for four bins of which those of i's set bits are kept: selectors of the first two and of the last two, and to
                     // get to the bytes behind theirs: bits to shift by once whole words have been left out, ~0 if one has to be
    uint4 keep[16];  // ~0 where the bin is kept
    // Each wave writes all of it, the same values, before it reads them: no barrier is needed.
    __device__ __forceinline__ void fill(int lane)
    {
        const uint32_t i = (uint32_t)lane & 15u, b0 = i & 1u, b1 = (i >> 1) & 1u, b2 = (i >> 2) & 1u, b3 = i >> 3, r2 = b0 + b1, r3 = r2 + b2, n = r3 + b3;
        auto half = [](uint32_t kept, uint32_t rank) __attribute__((always_inline)) { return kept ? 0x0100u + rank * 0x0202u : 0x0C0Cu; };  // 12: zero
        if (lane < 16) {
            pick[i] = make_uint4(half(b0, 0u) | half(b1, b0) << 16, half(b2, r2) | half(b3, r3) << 16, 16u * (n < 2u ? n : n - 2u), n < 2u ? 0u : ~0u);
            keep[i] = make_uint4(0u - b0, 0u - b1, 0u - b2, 0u - b3);
        }
        __builtin_amdgcn_wave_barrier();
    }
};
struct ByteWindow {
    uint32_t mask, rel, after;  // rel: bit position of the first code inside the window; after: the word behind the wave's last window
    uint32_t w[4];
    // run: kept bins of the record before these.  All lanes call this, with neighbouring stretches.
    __device__ __forceinline__ void fetch(const uint8_t* record, uint32_t W, int final, uint32_t run, uint32_t)
    {
        const int first = window_first(16u * run, final, 4);
        rel = 16u * run - 32u * (uint32_t)first;
        __builtin_memcpy(w, record + (uint32_t)(4 * (first + 4 + (int)W)), sizeof(w));
        const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)(run + (uint32_t)__popc(mask)), 63);
        const int word = code_word(16u * end, final > 0 ? final : 0);
        after = scalar_load(reinterpret_cast<const uint32_t*>(record) + (final < 0 ? 0 : 4 + (int)W + word));
    }
    template <typename Put>
    __device__ __forceinline__ void unpack(uint32_t, uint32_t, int shift, uint32_t base, const ByteTable* table, Put&& put)
    {
        while (__any(rel >= 32u)) {  // windows moved back from a record's end
            const bool on = rel >= 32u;
#pragma unroll
            for (int i = 0; i < 3; ++i) w[i] = on ? w[i + 1] : w[i];
            w[3] = on ? 0u : w[3];
            rel = on ? (rel < 128u ? rel - 32u : 0u) : rel;
        }
        const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp((int)after, (int)w[0], 0x130, 0xF, 0xF, false);  // the next lane's first word
        uint32_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_alignbit(i < 3 ? w[i + 1] : next, w[i], rel);
        uint32_t zeros = 0;  // top bits of the bytes whose other seven are all zero
#pragma unroll
        for (int i = 0; i < 4; ++i) zeros |= ~((v[i] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) & 0x80808080u;
        const uint4 pick = table->pick[mask & 15u], pick2 = table->pick[(mask >> 4) & 15u];
        uint32_t u[3];  // the words that the second four bins' bytes start in
#pragma unroll
        for (int i = 0; i < 3; ++i) u[i] = (v[i] & ~pick.w) | (v[i + 1] & pick.w);
        const uint32_t u0 = (uint32_t)(((uint64_t)u[1] << 32 | u[0]) >> pick.z), u1 = (uint32_t)(((uint64_t)u[2] << 32 | u[1]) >> pick.z);
        const uint32_t two[4] = {__builtin_amdgcn_perm(v[1], v[0], pick.x), __builtin_amdgcn_perm(v[1], v[0], pick.y),
                                 __builtin_amdgcn_perm(u1, u0, pick2.x), __builtin_amdgcn_perm(u1, u0, pick2.y)};
        constexpr uint32_t kMost = 0x7Fu << 20;  // the largest code's place
        if (shift == 20 && base < 0x80000000u - kMost && !__any(zeros)) {
            const uint4 keep = table->keep[mask & 15u], keep2 = table->keep[(mask >> 4) & 15u];
            const uint32_t bases[8] = {base & keep.x,  base & keep.y,  base & keep.z,  base & keep.w,
                                       base & keep2.x, base & keep2.y, base & keep2.z, base & keep2.w};
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                auto value = [&](uint32_t top) __attribute__((always_inline)) {
                    return __uint_as_float(((uint32_t)((int)top >> 4) & (0x80000000u | kMost)) + bases[j]);
                };
                put(j, make_float2(value(two[j >> 1] << (24 - 16 * (j & 1))), value(two[j >> 1] << (16 - 16 * (j & 1)))));
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                put(j, make_float2(__uint_as_float(dequantize_field(two[j >> 1], 16u * (j & 1), 8u, base, shift)),
                                   __uint_as_float(dequantize_field(two[j >> 1], 16u * (j & 1) + 8u, 8u, base, shift))));
        }
    }
};
// WIDEST: bits of a bin at most (16: codes of up to 8, 30: of up to 15); kByteCodes: the codes are bytes
constexpr int kByteCodes = 8;
template <int WIDEST>
struct PeerWindow : Stretch<8, WIDEST> {
    using Base = Stretch<8, WIDEST>;
    __device__ __forceinline__ void fetch(const uint8_t* record, uint32_t W, int final, uint32_t run, uint32_t twoN)
    {
        Base::fetch(reinterpret_cast<const uint32_t*>(record) + 4 + W, final, run * twoN);
    }
    template <typename Put>
    __device__ __forceinline__ void unpack(uint32_t twoN, uint32_t bits, int shift, uint32_t base, const ByteTable*, Put&& put)
    {
        Base::unpack(twoN, bits, shift, base, put);
    }
};
template <>
struct PeerWindow<kByteCodes> : ByteWindow {
};
template <int WIDEST>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_decode_peers(PeerList recs, uint32_t npeers, size_t S, uint32_t B, uint32_t W, int bits, int m,
                                                     uint32_t Tn, size_t C, const uint32_t* __restrict__ gprefix, float2* __restrict__ spec,
                                                     uint32_t sstride, bool vec, int pair_log)
{
    // sixteen slots and a gap, so that lanes sixteen slots apart use different banks
    constexpr int GAP = 2;
    __shared__ __align__(16) float2 stage[kTile + kTile / 16 * GAP];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t c = blockIdx.x / Tn;
    const uint32_t tile = blockIdx.x % Tn, tbase = tile * kTile, j0 = (uint32_t)tid * 8u;  // j0: this lane's first bin in the tile
    const uint32_t G = (W + GROUP_WORDS - 1) / GROUP_WORDS, g = tile * (kTile / 32 / GROUP_WORDS) + wave;
    const uint32_t byte = (tbase + j0) >> 3, twoN = 2u * (uint32_t)bits;
    const int shift = 23 - m, final = last_code_word((uint32_t)S, W);
    const bool in = byte < 4u * W;
    auto record_of = [&](uint32_t p) __attribute__((always_inline)) { return recs.p[p] + c * S; };
    auto flags_of = [&](uint32_t p) __attribute__((always_inline)) { return (uint32_t)record_of(p)[16u + (in ? byte : 0u)]; };
    auto run_of = [&](uint32_t p) __attribute__((always_inline)) { return scalar_load(gprefix + (p * C + c) * G + (g < G ? g : 0u)); };
    auto window = [&](PeerWindow<WIDEST>& o, uint32_t p, uint32_t flags, uint32_t run) __attribute__((always_inline)) {
        o.mask = in ? flags : 0u;
        const uint32_t n = (uint32_t)__popc(o.mask);
        o.fetch(record_of(p), W, final, run + wave_scan_incl(n) - n, twoN);
    };
    __shared__ __align__(16) ByteTable table;
    if constexpr (WIDEST == kByteCodes) table.fill(tid & 63);
    float2 acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = make_float2(0.f, 0.f);
    PeerWindow<WIDEST> o;
    uint32_t flags = flags_of(0u), run = run_of(0u);
    window(o, 0u, flags, run);
    const uint32_t last = npeers - 1u;
    flags = flags_of(last ? 1u : 0u);
    run = run_of(last ? 1u : 0u);
    auto add = [&](uint32_t p) __attribute__((always_inline)) {
        const uint32_t base = (scalar_load(reinterpret_cast<const uint32_t*>(record_of(p))) - 1u) << shift;
        o.unpack(twoN, (uint32_t)bits, shift, base, &table, [&](int j, float2 z) __attribute__((always_inline)) {
            acc[j] = make_float2(acc[j].x + z.x, acc[j].y + z.y);
        });
    };
    for (uint32_t p = 0; p < last; ++p) {
        PeerWindow<WIDEST> next;
        window(next, p + 1u, flags, run);
        const uint32_t after = p + 1u < last ? p + 2u : last;
        flags = flags_of(after);
        run = run_of(after);
        add(p);
        o = next;
    }
    add(last);
    // a tile is whole runs, and eight bins lie in one half of one of them: upwards two slots apart, or downwards
    auto gapped = [](uint32_t slot) __attribute__((always_inline)) { return slot + (slot >> 4) * GAP; };
    const uint32_t N1 = 1u << pair_log, half = N1 / 2, k1 = j0 & (N1 - 1u), start = j0 - k1;
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j) {
        uint32_t slot = j0 + j;
        if (pair_log) slot = start + (k1 < half ? 2u * (k1 + j) : (k1 + j == half ? 1u : 2u * (N1 - k1 - j) + 1u));
        stage[gapped(slot)] = acc[j];
    }
    __syncthreads();
    float2* X = spec + c * (size_t)sstride + tbase;
    const uint32_t count = units_in_tile<false>(0, c, B, tbase);
    if (vec) {
        float4* dst = reinterpret_cast<float4*>(X);  // the last one may reach past the chunk's last bin into the padding
#pragma unroll
        for (int i = 0; i < kTile / 2 / NT; ++i) {
            const uint32_t idx = (uint32_t)(tid + i * NT);
            if (2u * idx < count) dst[idx] = *reinterpret_cast<const float4*>(stage + gapped(2u * idx));
        }
    } else {
        for (uint32_t i = tid; i < count; i += NT) X[i] = stage[gapped(i)];
    }
}

// The widest codes, 16 bits and 32.
template <int NL>
__global__ __launch_bounds__(NT) void k_decode_peers_wide(PeerList recs, uint32_t npeers, size_t S, uint32_t B, uint32_t W, int bits,
                                                     int m, uint32_t Tn, size_t C, const uint32_t* __restrict__ gprefix,
                                                     float2* __restrict__ spec, uint32_t sstride, bool vec, int pair_log)
{
    __shared__ __align__(16) uint8_t windows[NL ? 4 * kWindow<NL> : 16];
    __shared__ __align__(16) float2 stage[kTile];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t c = blockIdx.x / Tn;
    const uint32_t tile = blockIdx.x % Tn, tbase = tile * kTile, row0 = (uint32_t)wave * WAVE_BINS;
    const uint32_t G = (W + GROUP_WORDS - 1) / GROUP_WORDS;
    uint8_t* window = windows + (NL ? wave * kWindow<NL> : 0);
    float2 acc[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = make_float2(0.f, 0.f);
    for (uint32_t p = 0; p < npeers; ++p) {
        const uint8_t* record = recs.p[p] + c * S;
        WaveCodes<NL> wc;
        const uint32_t g = tile * (kTile / 32 / GROUP_WORDS) + wave;
        uint32_t run, kept;
        fetch_flags<NL>(record, W, g, lane, wc);
        group_run(gprefix + (p * C + c) * G, W, g, run, kept);
        fetch_codes<NL, 2>(record, S, W, bits, run, kept, lane, wc);
        unpack_codes<NL, false>(wc, record, S, W, bits, 23 - m, lane, window, [&](int r, const float2& v) {
            acc[r] = make_float2(acc[r].x + v.x, acc[r].y + v.y);
        });
    }
    place_units(stage, row0, lane, pair_log, acc);
    __syncthreads();
    tile_from_lds(spec + c * (size_t)sstride + tbase, stage, units_in_tile<false>(0, c, B, tbase), vec, tid);
}

}  // namespace

// control block and histograms are adjacent: one fill
hipError_t launch_zero_control(uint8_t* ws_base, const Workspace& w, size_t C, hipStream_t s)
{
    uint32_t* status = reinterpret_cast<uint32_t*>(ws_base + w.status);
    const size_t zero_words = (w.hist - w.status) / 4 + C * kHistBins;
    FFTSP_LAUNCH("zero_fill", k_zero_u32, dim3((unsigned)((zero_words + 255) / 256)), dim3(256), 0, s, status,
                 zero_words);
    return hipGetLastError();
}

static Shape shape_of(const CodecArgs& a)
{
    const uint32_t B = codec_bins(a.L, a.time_domain);
    return Shape{B, codec_tiles(a.L, a.time_domain), (B + 31) / 32, a.k, a.sstride, a.word3, a.S, a.pair_log};
}
// chunks and tiles of a launch; the longest chunk's tiles
struct Extent {
    size_t chunks, tiles;
    uint32_t most;
};
static Extent extent_of(const CodecArgs& a)
{
    if (!a.tab) {
        const uint32_t Tn = codec_tiles(a.L, a.time_domain);
        return Extent{a.C, a.C * Tn, Tn};
    }
    Extent x{a.tab->count, ((size_t)a.tab->units << (kLongUnitLog - 11)) + a.tab->count, 0};
    for (uint32_t i = 0; i < a.tab->count; ++i) x.most = std::max(x.most, (1u << a.tab->tab.t[i].logM) / (uint32_t)kTile + 1u);
    return x;
}

// Short calls are bound by their launches, so the ones of one workgroup per chunk are left out there, and what they would
// find is found by every workgroup of the kernel behind them.
// In k_collect that is 16 KB more to read per tile.  Compress, chunks of 2^16: 16 tiles 30.5 -> 28.8 us, 512 39.7 -> 38.4,
// 1088 no difference, 2176 58.0 -> 58.9.
static bool find_in_collect(const Extent& x) { return x.tiles <= 1024; }
// k_emit finds the threshold itself, every workgroup all of it, where the launch saved weighs more.  Senders in us, k_resolve /
// without: chunks of 2^16 (17 tiles) 68 tiles 24.3 / 22.7, 374 34.0 / 32.5, 782 40.7 / 40.5, 1088 47.7 / 47.9;  2^17 (33) 66 23.8 / 22.3,
// 528 34.4 / 33.9, 1056 46.7 / 47.2;  2^18 (65) 65 25.4 / 24.3, 390 34.4 / 34.1, 520 36.4 / 37.2.  Binary16: 2^15 (9 tiles) 63 29.7 / 28.2, 495 33.8 / 32.1;
// 2^16 493 35.5 / 34.1;  2^18 260 30.0 / 29.5, 455 34.1 / 34.4.  Tensors: 2^16 493 38.9 / 37.5;  2^17 495 38.9 / 37.6;  2^18 65 28.3 / 27.1, 455 41.2 / 40.9.
// Top-k: 2^16 (32) 64 34.5 / 32.8, 512 36.1 / 35.2;  2^17 (64) 64 35.1 / 33.9, 256 35.5 / 34.3, 384 36.4 / 36.4, 512 37.0 / 36.9; but where the threshold's
// bucket is crowded and tiles have more candidates than are held (30 % of normal samples), 2^16 64 37.7 / 35.9, 512 39.8 / 39.1;  2^17 64 38.4 /
// 39.2, 256 39.5 / 40.9, 384 40.2 / 42.6, 512 40.2 / 42.9.  So long chunks of samples leave off earlier.
static bool resolve_in_emit(const Extent& x, int time_domain)
{
    return x.most <= kMergedTiles && x.tiles <= (time_domain && x.most > 32 ? 256 : 512);
}
// In k_decode it is the bitmap up to the tile, at most 256 bytes for each tile of the chunk, to read beside the tile's codes.
// Decompress: one chunk of 2^16 21.7 -> 17.7 us, 2^23 samples in chunks of 2^20 (2056 tiles) 49.4 -> 48.8, 2^24 76.6 -> 77.8, one
// chunk of 2^22 (1025 tiles) 50.3 -> 52.5.  Chunks of a few tiles always: Top-k of 2^24 samples in chunks of 2^12 32.8 -> 16.2.
static bool prefix_in_decode(const Extent& x) { return x.most <= 8 || (x.most <= 257 && x.tiles <= 4096); }

hipError_t launch_encode(const float* spec, const CodecArgs& a, uint8_t* stream_base, uint8_t* records,
                         uint8_t* ws_base, const Workspace& w, int hist_ready, hipStream_t s)
{
    const Shape u = shape_of(a);
    const Extent x = extent_of(a);
    const float2* X = reinterpret_cast<const float2*>(spec);
    const uint32_t* Xh = reinterpret_cast<const uint32_t*>(spec);
    uint32_t* hist = reinterpret_cast<uint32_t*>(ws_base + w.hist);
    uint32_t* sel = reinterpret_cast<uint32_t*>(ws_base + w.sel);
    uint32_t* tinfo = reinterpret_cast<uint32_t*>(ws_base + w.tinfo);
    uint32_t* tscan = reinterpret_cast<uint32_t*>(ws_base + w.tscan);
    uint2* cand = reinterpret_cast<uint2*>(ws_base + w.cand);
    if (x.tiles > 0x7fffffffu || x.most > (uint32_t)MAX_TILES) return hipErrorInvalidValue;
    if (a.time_domain && (a.tab || a.pair_log || hist_ready)) return hipErrorInvalidValue;
    // binary16 spectra come from the two-pass FFT only, which also fills the histogram
    if (a.half && (a.tab || a.time_domain || !a.pair_log || !hist_ready)) return hipErrorInvalidValue;
    if (a.tab && !hist_ready) return hipErrorInvalidValue;

    const bool window = a.time_domain && sampled(u.Tn, x.tiles, a.n % a.L == 0);
    if (window) {
        const auto sample = sample_stretch(a.L) == 8 ? k_sample<1> : k_sample<2>;
        FFTSP_LAUNCH("sample", sample, dim3((unsigned)a.C), dim3(kSampleLanes), 0, s, spec, a.L, a.k, a.n, sel, reinterpret_cast<uint32_t*>(ws_base + w.status));
    } else if (!hist_ready) {
        hipError_t e = launch_zero_control(ws_base, w, a.C, s);
        if (e != hipSuccess) return e;
        const uint32_t groups = (u.Tn + HIST_TILES - 1) / HIST_TILES;
        const uint32_t sgroups = (u.Tn + kHistSampleTiles - 1) / kHistSampleTiles;
        if (a.time_domain)
            FFTSP_LAUNCH("hist", k_hist_samples, dim3((unsigned)(a.C * sgroups)), dim3(NT), 0, s, spec, a.L, sgroups,
                         hist, a.n);
        else
            FFTSP_LAUNCH("hist", k_hist, dim3((unsigned)(a.C * groups)), dim3(NT), 0, s, X, a.sstride, a.pair_log, u.B,
                         groups, hist);
    }
    HeaderInfo h{a.write_header, a.hdr_n, a.hdr_L, a.hdr_C, (uint32_t)a.bits, (uint32_t)a.m, a.hdr_k, a.hdr_S,
                 a.hdr_theta, a.time_domain ? 1u : 0u, (uint32_t)a.hdr_scale};
    const uint32_t codes_per_bin = a.time_domain ? 1u : 2u;
    const dim3 per_tile((unsigned)x.tiles), per_chunk((unsigned)x.chunks);
    const bool merged = resolve_in_emit(x, a.time_domain);
    uint8_t* clear = merged ? records : nullptr;
    const ResolveArgs ra{a.bits, a.m, a.static_vmax, codes_per_bin};
    auto select = [&](auto table) {
        constexpr bool TABLE = decltype(table)::value;
        const TableArg<TABLE> tab = table_arg<TABLE>(a.tab);
        auto collect = [&](auto find) {
            constexpr bool FIND = decltype(find)::value;
            if constexpr (TABLE) {
                FFTSP_LAUNCH("collect", (k_collect<FIND, true, false, false>), per_tile, dim3(NT), 0, s, X, u, hist, sel, tinfo, tscan, cand, clear, tab, a.n);
            } else {
                if (a.time_domain)
                    FFTSP_LAUNCH("collect", (k_collect<FIND, false, true, false>), per_tile, dim3(NT), 0, s, spec, u, hist, sel, tinfo, tscan, cand, clear, tab, a.n);
                else if (a.half)
                    FFTSP_LAUNCH("collect", (k_collect<FIND, false, false, true>), per_tile, dim3(NT), 0, s, Xh, u, hist, sel, tinfo, tscan, cand, clear, tab, a.n);
                else
                    FFTSP_LAUNCH("collect", (k_collect<FIND, false, false, false>), per_tile, dim3(NT), 0, s, X, u, hist, sel, tinfo, tscan, cand, clear, tab, a.n);
            }
        };
        if (window) {
            if constexpr (!TABLE)
                FFTSP_LAUNCH("collect", (k_collect<false, false, true, false, true>), per_tile, dim3(NT), 0, s, spec, u, hist, sel, tinfo, tscan, cand, clear, tab,
                             a.n);
        } else if (find_in_collect(x)) {
            collect(std::true_type{});
        } else {
            FFTSP_LAUNCH("find_bucket", k_find_bucket<TABLE>, per_chunk, dim3(NT), 0, s, hist, u, sel, tab);
            collect(std::false_type{});
        }
        if (merged) return hipGetLastError();
        const bool counted = x.most > kKeptTiles;
        if (counted) {
            LongStarts at{};
            uint32_t parts = (uint32_t)x.chunks * parts_of(x.most);
            if constexpr (TABLE) {
                // the longest tensors are the last ones
                parts = 0;
                at.first = a.tab->count;
                while (at.first > 0 && (1u << a.tab->tab.t[at.first - 1].logM) / (uint32_t)kTile + 1u > kFewTiles) --at.first;
                for (uint32_t i = at.first; i < a.tab->count; ++i) {
                    at.at[at.count++] = (uint16_t)parts;
                    parts += parts_of((1u << a.tab->tab.t[i].logM) / (uint32_t)kTile + 1u);
                }
            }
            FFTSP_LAUNCH("count_digit", k_count_digit<TABLE>, dim3(parts), dim3(NT), 0, s, u, tinfo, tscan, cand, tab, at);
            FFTSP_LAUNCH("mark", k_mark<TABLE>, dim3(parts), dim3(NT), 0, s, u, sel, tinfo, tscan, cand, tab, at);
        }
        auto resolve = [&](auto waves, auto fetch) {
            constexpr int NW = decltype(waves)::value, FETCH = decltype(fetch)::value;
            if constexpr (!TABLE) {
                if (window) {
                    FFTSP_LAUNCH("resolve", (k_resolve<false, true, NW, FETCH>), per_chunk, dim3(NW * 64), 0, s, u, ra, sel, tinfo, tscan, cand, records,
                                 stream_base, h, tab, spec, a.n);
                    return hipGetLastError();
                }
            }
            FFTSP_LAUNCH("resolve", (k_resolve<TABLE, false, NW, FETCH>), per_chunk, dim3(NW * 64), 0, s, u, ra, sel, tinfo, tscan, cand, records, stream_base,
                         h, tab, nullptr, a.n);
            return hipGetLastError();
        };
        // few waves for few tiles: their barriers are cheaper than more hands
        constexpr std::integral_constant<int, kFetch> some{};
        if (x.most <= 40u) return resolve(std::integral_constant<int, 4>{}, some);
        if (x.most <= kHeldTiles<8, kFetch>) return resolve(std::integral_constant<int, 8>{}, some);
        if (x.most <= kFewTiles || counted) return resolve(std::integral_constant<int, 16>{}, some);
        return resolve(std::integral_constant<int, 16>{}, std::integral_constant<int, kFetchMost>{});
    };
    const hipError_t e = a.tab ? select(std::true_type{}) : select(std::false_type{});
    if (e != hipSuccess) return e;
#define FFTSP_EMIT_AS(TABLE, REAL, HALF, MERGED, src, lds)                                                                          \
    FFTSP_LAUNCH("emit", (k_emit<TABLE, REAL, HALF, MERGED>), per_tile, dim3(NT), lds, s, src, u, emit_reversed(per_tile.x), ra, sel, tscan, tinfo, cand, records, \
                 stream_base, h, table_arg<TABLE>(a.tab), a.n)
#define FFTSP_EMIT(TABLE, REAL, HALF, src)                              \
    if (merged)                                                         \
        FFTSP_EMIT_AS(TABLE, REAL, HALF, true, src, 0);     \
    else                                                                \
        FFTSP_EMIT_AS(TABLE, REAL, HALF, false, src, 0)
    if (a.tab) {
        FFTSP_EMIT(true, false, false, X);
    } else if (a.time_domain) {
        FFTSP_EMIT(false, true, false, spec);
    } else if (a.half) {
        FFTSP_EMIT(false, false, true, Xh);
    } else {
        FFTSP_EMIT(false, false, false, X);
    }
#undef FFTSP_EMIT
#undef FFTSP_EMIT_AS
    return hipGetLastError();
}

hipError_t launch_decode(const uint8_t* stream_base, const uint8_t* records, const CodecArgs& a, float* spec,
                         uint8_t* ws_base, const Workspace& w, int check_header, uint32_t* verdicts, const StatusNote* first,
                         hipStream_t s)
{
    const Shape u = shape_of(a);
    const Extent x = extent_of(a);
    uint32_t* ctl = first ? reinterpret_cast<uint32_t*>(ws_base + w.status) : nullptr;
    const StatusNote note = first ? *first : StatusNote{};
    if (x.tiles > 0x7fffffffu) return hipErrorInvalidValue;
    if (a.half && (a.tab || a.time_domain)) return hipErrorInvalidValue;
    if (a.time_domain && (a.tab || a.pair_log)) return hipErrorInvalidValue;
    HeaderInfo h{check_header, a.hdr_n, a.hdr_L, a.hdr_C, (uint32_t)a.bits, (uint32_t)a.m, a.hdr_k, a.hdr_S,
                 a.hdr_theta, a.time_domain ? 1u : 0u, (uint32_t)a.hdr_scale};
    uint32_t* gprefix = nullptr;
    if (!prefix_in_decode(x)) {
        gprefix = reinterpret_cast<uint32_t*>(ws_base + w.prefix);
        const uint32_t parts = prefix_parts(a.tab ? (1u << a.tab->tab.t[a.tab->count - 1].logM) / 32u + 1u : u.W);  // of the longest chunk
        if (a.tab)
            FFTSP_LAUNCH("group_prefix", k_group_prefix<true>, dim3((unsigned)x.chunks * parts), dim3(RT), 0, s, stream_base, records, u, h,
                         parts, gprefix, verdicts, ctl, note, table_arg<true>(a.tab));
        else
            FFTSP_LAUNCH("group_prefix", k_group_prefix<false>, dim3((unsigned)x.chunks * parts), dim3(RT), 0, s, stream_base, records, u, h,
                         parts, gprefix, verdicts, ctl, note, table_arg<false>(a.tab));
    }
    const bool vec = a.tab || (a.sstride == padded_bins(a.L) && (reinterpret_cast<uintptr_t>(spec) & 15u) == 0);
#define FFTSP_DECODE_AS(NL, TABLE, REAL, HALF, T)                                                                          \
    if (gprefix)                                                                                                           \
        FFTSP_DECODE_WITH(NL, false, TABLE, REAL, HALF, T);                                                                \
    else                                                                                                                   \
        FFTSP_DECODE_WITH(NL, true, TABLE, REAL, HALF, T)
#define FFTSP_DECODE_WITH(NL, COUNT, TABLE, REAL, HALF, T)                                                                 \
    FFTSP_LAUNCH("decode", (k_decode<NL, COUNT, TABLE, REAL, HALF>), dim3((unsigned)x.tiles), dim3(NT), 0, s, stream_base, records, u, \
                 a.bits, a.m, gprefix, h, verdicts, ctl, note, reinterpret_cast<T*>(spec), vec, table_arg<TABLE>(a.tab), a.n)
#define FFTSP_DECODE(NL)                                       \
    do {                                                       \
        if (a.tab) {                                           \
            FFTSP_DECODE_AS(NL, true, false, false, float2);   \
        } else if (a.half) {                                   \
            FFTSP_DECODE_AS(NL, false, false, true, uint32_t); \
        } else {                                               \
            FFTSP_DECODE_AS(NL, false, false, false, float2);  \
        }                                                      \
    } while (0)
    // code widths are 3..16 or 32 bits; the codes of a wave's 512 units are at most 1 KiB for 16 bits a unit, else 2 KiB
    if (a.time_domain && a.bits <= 16) {
        FFTSP_DECODE_AS(1, false, true, false, float);
    } else if (a.time_domain) {
        FFTSP_DECODE_AS(0, false, true, false, float);
    } else if (a.bits <= 8) {
        FFTSP_DECODE(1);
    } else if (a.bits <= 16) {
        FFTSP_DECODE(2);
    } else {
        FFTSP_DECODE(0);
    }
#undef FFTSP_DECODE_WITH
#undef FFTSP_DECODE_AS
#undef FFTSP_DECODE
    return hipGetLastError();
}

hipError_t launch_decode_peers(const PeerList& streams, int npeers, const CodecArgs& a, float* spec, uint8_t* ws_base,
                               const Workspace& w, const PeerWorkspace& pw, hipStream_t s)
{
    const Shape u = shape_of(a);
    uint32_t* ctl = reinterpret_cast<uint32_t*>(ws_base + w.status);
    uint32_t* gprefix = reinterpret_cast<uint32_t*>(ws_base + pw.prefix);
    uint32_t* verdicts = reinterpret_cast<uint32_t*>(ws_base + pw.verd);
    if (npeers < 1 || npeers > kMaxPeers || a.half || a.tab || a.time_domain) return hipErrorInvalidValue;
    const size_t count = a.C * (size_t)npeers;
    if (a.C * (size_t)u.Tn > 0x7fffffffu || count > 0x7fffffffu) return hipErrorInvalidValue;
    HeaderInfo h{1, a.hdr_n, a.hdr_L, a.hdr_C, (uint32_t)a.bits, (uint32_t)a.m, a.hdr_k, a.hdr_S, a.hdr_theta, 0u, 0u};
    const uint32_t parts = prefix_parts(u.W);
    if (count * parts > 0x7fffffffu) return hipErrorInvalidValue;
    FFTSP_LAUNCH("group_prefix", k_group_prefix_peers, dim3((unsigned)(count * parts)), dim3(RT), 0, s, streams, (uint32_t)a.C, a.S, u.W,
                 a.k, h, parts, gprefix, verdicts, ctl, status_note(count, pw.verd));
    PeerList recs{};
    for (int i = 0; i < npeers; ++i) recs.p[i] = streams.p[i] + 64;  // records follow the 64-byte stream header
    const bool vec = a.sstride == padded_bins(a.L) && (reinterpret_cast<uintptr_t>(spec) & 15u) == 0;
#define FFTSP_DECODE_PEERS(kern)                                                                                       \
    FFTSP_LAUNCH("decode", kern, dim3((unsigned)(a.C * u.Tn)), dim3(NT), 0, s, recs, (uint32_t)npeers, a.S, u.B, u.W, a.bits, a.m, u.Tn, a.C, \
                 gprefix, reinterpret_cast<float2*>(spec), a.sstride, vec, a.pair_log)
    if (a.bits == 8)
        FFTSP_DECODE_PEERS(k_decode_peers<kByteCodes>);
    else if (a.bits < 8)
        FFTSP_DECODE_PEERS(k_decode_peers<16>);
    else if (a.bits <= 15)
        FFTSP_DECODE_PEERS(k_decode_peers<30>);
    else if (a.bits <= 16)
        FFTSP_DECODE_PEERS(k_decode_peers_wide<2>);
    else
        FFTSP_DECODE_PEERS(k_decode_peers_wide<0>);
#undef FFTSP_DECODE_PEERS
    return hipGetLastError();
}

}  // namespace fftsp

// Chunk-resident codec: chunks of up to 2^15 samples go through the whole sender, or the whole receiver, in one
// workgroup, so that a gradient is read once and only the packed record is written (and the other way round).
//
// A chunk of L = 2M samples (M = 2^LOGM complex points, LOGM = 4 .. 14) is at most 128 KiB of complex values, which
// fits the LDS of a compute unit together with a 16 KiB twiddle table.  The sender is
//     samples -> first FFT stage in registers -> LDS stages -> real-FFT split into registers
//     -> exact radix select on the registers -> ranks from ballots -> Algorithm 1 -> record image in LDS -> memory
// and the receiver
//     record image -> LDS -> (word, prefix) table of the bitmap -> dequantised bins in registers -> LDS
//     -> inverse split -> first inverse stage in registers -> LDS stages -> last stage straight to memory.
// Between the two ends nothing leaves the workgroup: no spectrum, no histogram and no candidate list in memory, and one
// launch where the per-tile kernels (codec.hip) take ten.  The transform's arithmetic is that of fft_core.h.
//
// What bounds it: vector instruction issue (chunks of 2^12, 10-bit codes of 15 % of the bins: 114 instructions per bin sending, more than
// half of them transform and split, 101 receiving; the vector units are busy 30 to 59 and 33 to 65 % of the time, at two to four
// cycles an instruction), the barriers between its stages and, for the longest chunks, the
// few waves one workgroup per compute unit leaves.  Measured on 25.6 M samples, compress + decompress, against the per-tile kernels
// with their ten sweeps and 16 KiB of histogram per chunk: L = 2^12 636 -> 98 us, one chunk of 2^10 91 -> 22 us.
//
// A workgroup holds 2^LOGE complex points, i.e. one chunk, or several when they are short.  Every chunk belongs to a
// group of WAVES waves.  Up to M = 1024 that is a single wave: waves then share nothing but the twiddle table and run
// without a workgroup barrier.
#include "chunk.h"
#include "codec_core.h"
#include "fft_core.h"
#include "receive.h"
#include "receive_table.h"
#include "short.h"
#include "short_core.h"
#include "split_tile.h"

#include <type_traits>

namespace fftsp {
namespace {

// every LOGM there is
#define FFTSP_CHUNK_SIZES(X) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14)

struct GroupScratch {
    uint32_t bucket, need, count, listed;
    uint32_t a[16], b[16], v[16];
};
static_assert(sizeof(GroupScratch) % 16 == 0, "the LDS regions behind it stay aligned");

// Coarse twiddles (steps of 1/2048 of a turn, or of 1/R for R < 2048) that the stages of an R-point transform look up: those
// of the last part of the turn are never wanted, and what they would take decides how many workgroups a compute unit holds.
// At R = 2048 they are half a turn, the other half their negatives: 1024 entries beside 32 KB of data are a quarter of a compute
// unit's LDS to the byte.  25 M samples in chunks of 2^12, three workgroups a compute unit -> four: sender 66 -> 58 us, receiver 53 -> 47.
constexpr bool half_turn(int logr) { return logr == 11; }
constexpr int coarse_twiddles(int logr)
{
    if (half_turn(logr)) return 1 << (logr - 1);
    int most = 0;
    for (int ns = 0; ns < logr;) {
        const int rl = stage_radix_log(logr - ns), at = ((1 << rl) - 1) * ((1 << ns) - 1) << (logr - ns - rl);
        most = at > most ? at : most;
        ns += rl;
    }
    return ((most >> (logr > 11 ? logr - 11 : 0)) + 2) & ~1;  // whole 16 bytes
}
template <int LOGM, int NTHREADS>
struct Geo {
    static constexpr int M = 1 << LOGM;
    // 16 points per lane; 8 at M = 2^9, so that a wave still has one chunk
    static constexpr int LOGE = LOGM > 12 ? LOGM : (LOGM == 9 ? 11 : 12), E = 1 << LOGE;
    static constexpr int NT = NTHREADS, NW = NT / 64;
    static constexpr int T = E / M;                            // chunks per workgroup
    static constexpr int WAVES = NW > T ? NW / T : 1;          // waves per chunk
    static constexpr int CPW = T > NW ? T / NW : 1;            // chunks a group takes one after the other
    static constexpr int GROUPS = NW / WAVES;
    static constexpr int NL = 64 * WAVES;                      // lanes per group
    static constexpr int R = M / NL > 1 ? M / NL : 1;          // rows of 64 bins per wave
    static constexpr int LR = M < 64 ? M : 64;                 // bins of a row that exist
    static constexpr int HB = M <= 256 ? 0 : (M <= 2048 ? 11 : 12);  // first radix digit; 0: bisection
    static constexpr int WC = M >= 32 ? M / 32 : 1;            // bitmap words of a chunk without the Nyquist bin's
    static constexpr int GROUP_WORDS = CPW * WC;                 // bitmap words of a group
    static constexpr int TW = coarse_twiddles(LOGM) + (LOGM <= 11 ? 0 : 1 << (LOGM - 11));  // entries of the stage twiddle table
    // LDS bytes of a group: its complex values, later its histogram, candidate list and record image
    static constexpr int DATA = E / GROUPS * 8, REGION = DATA > (4 << HB) ? DATA : (4 << HB);
    static constexpr int SCRATCH = GROUPS * (int)sizeof(GroupScratch) + 16;  // and the word the groups agree through
    // A sender's lies at the end of its groups' regions where histogram, list and image leave room.
    static constexpr int INSIDE = LOGM >= 11 ? (int)sizeof(GroupScratch) + 16 : 0;
    static constexpr int SENDER_FRONT = INSIDE ? 0 : SCRATCH;
    static constexpr int RECEIVER_FRONT = WC > 64 ? SCRATCH : 0;  // one wave counts a short bitmap
    // of a receiver's group: its record images and behind them the bitmap's words with their prefixes, later its complex values
    __host__ __device__ static constexpr size_t receiver_region(size_t images)
    {
        const size_t need = (images + GROUP_WORDS * 8 + 15) / 16 * 16;
        return need > (size_t)DATA ? need : (size_t)DATA;
    }
    // record image of one chunk of up to 16-bit codes, in words; short chunks keep theirs beside the data
    static constexpr int IMAGE = HB ? 0 : ((16 + 4 * (M / 32 + 1) + 4 * (M + 1) + 16) / 4 + 3) & ~3;
};
// measured: 8 points per lane beat 16 at M = 2^12 (twice the waves on the same LDS); above it the radix-16 first
// stage wants 16
template <int LOGM>
constexpr int uniform_threads()
{
    return LOGM <= 11 ? 256 : (LOGM <= 13 ? 512 : 1024);
}

// Orders LDS accesses among the waves of a group.  LDS operations of one wave complete in order, so within a wave
// it is the compiler alone that has to be held back.
template <int WAVES>
__device__ __forceinline__ void group_sync()
{
    if constexpr (WAVES == 1) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// Complex values of all chunks of a workgroup lie behind each other in LDS; the low four index bits are XORed with the
// next four, so that both "consecutive" accesses and the stride-8 and stride-16 ones of the first stages spread
// over all banks.
__device__ __forceinline__ constexpr int flat(int g) { return g ^ ((g >> 4) & 15); }
// flat(g + o) from flat(g), for a constant o that shares no bit with g: the XOR is linear, so the part of o above the
// low four bits is an address offset and only what it does to those bits costs an instruction (often nothing)
__device__ __forceinline__ int flat_plus(int flat_g, int o) { return (flat_g ^ (flat(o) & 15)) + (o & ~15); }

// ------------------------------------------------------------------- FFT ----
// Stage twiddles exp(-2 pi i e / R): what there are of R of them up to R = 2048; above it the coarse entries and the R / 2048
// fine ones behind them, multiplied where a stage needs the fine part (the last one).
template <int LOGR, int NT>
__device__ __forceinline__ void load_chunk_twiddles(float2* tw, const Tables& tb, int tid)
{
    constexpr int COUNT = coarse_twiddles(LOGR), ITERS = (COUNT + NT - 1) / NT;
    float2 v[ITERS];  // all loads before the first wait
#pragma unroll
    for (int i = 0; i < ITERS; ++i) {
        const int e = tid + i * NT < COUNT ? tid + i * NT : 0;
        v[i] = tb.hi[LOGR <= 11 ? e << (LOGR <= 11 ? 11 - LOGR : 0) : e];
    }
    if constexpr (LOGR > 11)
        if (tid < (1 << (LOGR - 11))) tw[COUNT + tid] = tb.lo[tid << (22 - LOGR)];
#pragma unroll
    for (int i = 0; i < ITERS; ++i)
        if (tid + i * NT < COUNT) tw[tid + i * NT] = v[i];
}
// most: the largest idx of any lane
template <int LOGR, int SHIFT>
__device__ __forceinline__ float2 stage_twiddle(const float2* tw, int idx, int most)
{
    constexpr int COARSE = coarse_twiddles(LOGR);
    if constexpr (half_turn(LOGR)) {
        if (most << SHIFT < COARSE) return tw[idx << SHIFT];
        const float2 c = tw[(idx << SHIFT) & (COARSE - 1)];
        const uint32_t sign = ((uint32_t)idx << (SHIFT + 32 - LOGR)) & 0x80000000u;
        return make_float2(__uint_as_float(__float_as_uint(c.x) ^ sign), __uint_as_float(__float_as_uint(c.y) ^ sign));
    } else if constexpr (LOGR <= 11)
        return tw[idx << SHIFT];
    else if constexpr (SHIFT >= LOGR - 11)
        return tw[idx << (SHIFT - (LOGR - 11))];
    else
        return cmul(tw[idx >> (LOGR - 11 - SHIFT)], tw[COARSE + ((idx << SHIFT) & ((1 << (LOGR - 11)) - 1))]);
}

// Butterfly q of a lane: transform b, index j.  A wave's butterflies are consecutive, so its points are too.
template <int LOGR, int LOGE, int NT, int RL>
struct Butterflies {
    static constexpr int PER = (1 << (LOGE - RL)) / NT, RHO = 1 << RL, STEP = 1 << (LOGR - RL);
    static_assert(PER >= 1, "every lane has work");
    static __device__ __forceinline__ int index(int tid, int q)
    {
        return (tid >> 6) * (64 * PER) + q * 64 + (tid & 63);
    }
    static __device__ __forceinline__ int j(int w) { return w & (STEP - 1); }
    static __device__ __forceinline__ int b(int w) { return w >> (LOGR - RL); }
};

template <int LOGR, int LOGE, int NT, bool INV, int NS_LOG, int RL>
__device__ __forceinline__ void stage_compute(float2 (&v)[(1 << (LOGE - RL)) / NT][1 << RL], const float2* tw, int tid)
{
    using B = Butterflies<LOGR, LOGE, NT, RL>;
#pragma unroll
    for (int q = 0; q < B::PER; ++q) {
        if constexpr (NS_LOG > 0) {
            const int k = B::j(B::index(tid, q)) & ((1 << NS_LOG) - 1);
#pragma unroll
            for (int t = 1; t < B::RHO; ++t) {
                const float2 c = stage_twiddle<LOGR, LOGR - NS_LOG - RL>(tw, t * k, t * ((1 << NS_LOG) - 1));
                v[q][t] = INV ? cmulc(v[q][t], c) : cmul(v[q][t], c);
            }
        }
        butterfly<RL, INV>(v[q]);
    }
}

// out(b, i, o, value) receives output i + o of transform b; o is a constant multiple of what i can reach
template <int LOGR, int LOGE, int NT, int NS_LOG, int RL, typename Out>
__device__ __forceinline__ void stage_outputs(const float2 (&v)[(1 << (LOGE - RL)) / NT][1 << RL], int tid, Out&& out)
{
    using B = Butterflies<LOGR, LOGE, NT, RL>;
#pragma unroll
    for (int q = 0; q < B::PER; ++q) {
        const int w = B::index(tid, q), j = B::j(w), b = B::b(w), k = j & ((1 << NS_LOG) - 1);
        const int base = ((j >> NS_LOG) << (NS_LOG + RL)) + k;
#pragma unroll
        for (int t = 0; t < B::RHO; ++t) out(b, base, t << NS_LOG, v[q][t]);
    }
}
template <int LOGR, int LOGE, int NT, int NS_LOG, int RL>
__device__ __forceinline__ void stage_to_lds(const float2 (&v)[(1 << (LOGE - RL)) / NT][1 << RL], float2* d, int tid)
{
    stage_outputs<LOGR, LOGE, NT, NS_LOG, RL>(v, tid, [&](int b, int i, int o, float2 z) {
        d[flat_plus(flat((b << LOGR) + i), o)] = z;
    });
}

// The stages from NS_LOG applied levels on, data in LDS and visible.  TO_LDS: the result goes back to d (visible to
// the group afterwards); otherwise the last stage hands every value to out (see stage_outputs).
template <int LOGR, int LOGE, int NT, int WAVES, bool INV, int NS_LOG, bool TO_LDS, typename Out>
__device__ __forceinline__ void fft_rest(float2* d, const float2* tw, int tid, Out&& out)
{
    if constexpr (NS_LOG < LOGR) {
        constexpr int RL = stage_radix_log(LOGR - NS_LOG);
        using B = Butterflies<LOGR, LOGE, NT, RL>;
        constexpr bool LAST = NS_LOG + RL == LOGR;
        float2 v[B::PER][B::RHO];
#pragma unroll
        for (int q = 0; q < B::PER; ++q) {
            const int w = B::index(tid, q), f = flat((B::b(w) << LOGR) + B::j(w));
#pragma unroll
            for (int t = 0; t < B::RHO; ++t) v[q][t] = d[flat_plus(f, t * B::STEP)];
        }
        stage_compute<LOGR, LOGE, NT, INV, NS_LOG, RL>(v, tw, tid);
        if constexpr (LAST && !TO_LDS) {
            stage_outputs<LOGR, LOGE, NT, NS_LOG, RL>(v, tid, out);
        } else {
            group_sync<WAVES>();
            stage_to_lds<LOGR, LOGE, NT, NS_LOG, RL>(v, d, tid);
            group_sync<WAVES>();
            if constexpr (!LAST) fft_rest<LOGR, LOGE, NT, WAVES, INV, NS_LOG + RL, TO_LDS>(d, tw, tid, out);
        }
    }
}

// first stage of an R-point transform: its inputs are v[q][t] = point j + t*R/RHO of transform b
template <int LOGR, int LOGE, int NT, int WAVES, bool INV, bool TO_LDS, int RL, typename Out>
__device__ __forceinline__ void fft_from_registers(float2 (&v)[(1 << (LOGE - RL)) / NT][1 << RL], float2* d, const float2* tw,
                                                   int tid, Out&& out)
{
    static_assert(RL == stage_radix_log(LOGR), "the plan's first radix");
    stage_compute<LOGR, LOGE, NT, INV, 0, RL>(v, tw, tid);
    if constexpr (RL == LOGR && !TO_LDS) {
        stage_outputs<LOGR, LOGE, NT, 0, RL>(v, tid, out);
    } else {
        stage_to_lds<LOGR, LOGE, NT, 0, RL>(v, d, tid);
        group_sync<WAVES>();
        fft_rest<LOGR, LOGE, NT, WAVES, INV, RL, TO_LDS>(d, tw, tid, out);
    }
}
struct NoOut {
    __device__ void operator()(int, int, int, float2) const {}
};

// Which chunks a workgroup holds in its T slots, and where their samples and records are.
// Uniform calls: chunks c0 .. c0+T-1 of a gradient cut into equal pieces.
struct UniformChunks {
    size_t first_sample, n, first_record, c0;
    uint32_t slots, chunk_len, S;  // slots: chunks from c0 on that exist
    int aligned;
    __device__ __forceinline__ UniformChunks(size_t n_, size_t C, uint32_t T, uint32_t L, uint32_t S_, int aligned_)
        : n(n_), c0((size_t)blockIdx.x * T), chunk_len(L), S(S_), aligned(aligned_)
    {
        first_sample = c0 * L;
        first_record = c0 * S;
        slots = C - c0 < (size_t)T ? (uint32_t)(C - c0) : T;
    }
    __device__ __forceinline__ bool exists(int b) const { return (uint32_t)b < slots; }
    __device__ __forceinline__ Span span(int b) const { return Span{first_sample + (size_t)((uint32_t)b * chunk_len), n}; }
    // all T slots hold whole chunks: the samples are one aligned run from first_sample on
    __device__ __forceinline__ bool whole(int T) const { return aligned && first_sample + (size_t)((uint32_t)T * chunk_len) <= n; }
    __device__ __forceinline__ size_t record(int b) const { return first_record + (size_t)((uint32_t)b * S); }
    __device__ __forceinline__ size_t verdict(int b) const { return c0 + (size_t)b; }
};
// Per-tensor calls: one tensor in the first slot of each group (spread over workgroups rather than packed: there are
// few of them, and it is their latency that counts).  A lane only ever asks for its own group's slots.
struct ListedChunk {
    size_t first_sample, first_record, number;
    uint32_t length;
    int slot;  // -1 if the group has none
    __device__ __forceinline__ ListedChunk(const TensorTable& t, const TensorPiece& piece, int group, int cpw)
    {
        const bool has = group < (int)piece.count;
        const uint32_t entry = (uint32_t)piece.first + (has ? (uint32_t)group : 0u);
        first_sample = t.goff[entry];
        first_record = t.roff[entry];
        length = t.glen[entry];
        number = (size_t)(t.base + entry);
        slot = has ? group * cpw : -1;
    }
    __device__ __forceinline__ bool exists(int b) const { return b == slot; }
    __device__ __forceinline__ Span span(int b) const
    {
        return exists(b) ? Span{first_sample, first_sample + length} : Span{0, 0};
    }
    __device__ __forceinline__ bool whole(int) const { return false; }
    __device__ __forceinline__ size_t record(int) const { return first_record; }
    __device__ __forceinline__ size_t verdict(int) const { return number; }
};

// Forward transform of the workgroup's chunks up to Z[k] in d, visible to the group.
// The stage twiddle table must have been filled before (the barrier for it is taken here, behind the loads).
template <typename G, int LOGM, typename Where>
__device__ __forceinline__ void forward_tile(const float* __restrict__ in, const Where& where, const Tables& tb, float2* d, const float2* tw, int tid)
{
    constexpr int RL = stage_radix_log(LOGM);
    using B = Butterflies<LOGM, G::LOGE, G::NT, RL>;
    float2 v[B::PER][B::RHO];
    if (where.whole(G::T)) {
        const float2* src = reinterpret_cast<const float2*>(in + where.first_sample);
#pragma unroll
        for (int q = 0; q < B::PER; ++q) {
            const int w = B::index(tid, q), g = (B::b(w) << LOGM) + B::j(w);
#pragma unroll
            for (int t = 0; t < B::RHO; ++t) v[q][t] = src[g + t * B::STEP];
        }
    } else {
#pragma unroll
        for (int q = 0; q < B::PER; ++q) {
            const int w = B::index(tid, q);
            load_pairs(v[q], in, where.span(B::b(w)), (uint32_t)G::M, (uint32_t)B::j(w), (uint32_t)B::STEP, tb);
        }
    }
    __syncthreads();
    fft_from_registers<LOGM, G::LOGE, G::NT, G::WAVES, false, true, RL>(v, d, tw, tid, NoOut());
}

// W_L^k for the even/odd split of a chunk of 2^(LOGM+1) samples
template <int LOGM>
__device__ __forceinline__ float2 split_twiddle(const Tables& tb, int k)
{
    if constexpr (LOGM <= 10)
        return tb.hi[k << (10 - LOGM)];
    else
        return cmul(tb.hi[k >> (LOGM - 10)], tb.lo[(k & ((1 << (LOGM - 10)) - 1)) << (21 - LOGM)]);
}
// X[k], 0 <= k < M, from Z[k] and Z[M-k]
template <int LOGM>
__device__ __forceinline__ float2 split_bin(float2 a, float2 b, int k, const Tables& tb)
{
    const float2 x = split_fwd(a, b, split_twiddle<LOGM>(tb, k));
    return k == 0 ? make_float2(a.x + a.y, 0.f) : x;
}
template <int LOGM>
__device__ __forceinline__ float2 nyquist_bin(const float2* d, int base)
{
    const float2 a = d[flat(base)];
    return make_float2(a.x - a.y, 0.f);
}

// --------------------------------------------------------- select and pack ----
// Packing a row of bins costs the same however few of them survive.  Where at most this many do, and the region has room behind
// the image, the survivors first move there, next to each other.
// Senders of 25 M normal samples, row by row -> next to each other, us, at 15 %, 30 %, 50 % kept.  Transforms, 10-bit codes: L = 2^11
// 51.8 -> 48.5, 52.5 -> 50.4, 53.3 -> 53.3;  2^12 55.5 -> 51.7, 56.3 -> 53.7, 57.0 -> 56.7;  2^13 61.1 -> 57.9, 63.0 -> 60.8, 64.0 -> 63.5;
// 2^15 86.7 -> 80.2, 87.6 -> 83.1, 89.9 -> 87.8; at 75 % none gains.  8-bit codes are stores and no atomics; at 15 %, 30 %, 40 %, 50 %: 2^11
// 48.0 -> 47.6, 48.9 -> 48.4, 48.6 -> 49.3, 49.3 -> 50.4;  2^12 51.3 -> 49.5, 51.4 -> 50.7, 51.2 -> 51.3, 52.4 -> 52.9;  2^13 57.7 -> 56.9, 58.7 ->
// 57.8, 58.7 -> 58.5, 58.1 -> 58.5;  2^15 81.5 -> 79.3, 82.1 -> 81.6, 83.3 -> 83.0, 83.2 -> 84.1.  Top-k, 10 bits, 15 %, 30 %, 50 %: 2^10 57.8 ->
// 52.6, 58.7 -> 55.4, 58.8 -> 59.1;  2^12 43.9 -> 38.5, 44.7 -> 41.0, 44.9 -> 45.6;  8-bit codes, 10 %, 20 %, 30 %: 2^10 51.3 -> 50.9, 51.6 -> 52.3,
// 52.8 -> 53.6;  2^12 38.6 -> 37.5, 38.6 -> 38.1, 39.4 -> 39.4;  2^15 66.4 -> 64.3, 66.5 -> 65.4, 67.2 -> 67.0.
template <bool REAL, int WAVES>
__host__ __device__ constexpr uint32_t most_packed(uint32_t units, int bits)
{
    if (bits == 32) return 0u;
    const bool several = !REAL && WAVES > 1;
    if (bits == 8) return several ? units * 2u / 5u : units / (REAL ? 5u : 3u);
    return units / (several ? 2u : 3u);
}
// Whether a kernel's survivors move.  Top-k has a kernel for each way: one that holds both is slower on either.
// Senders of 8-bit codes in us, no survivor moved anywhere -> one kernel -> two.  80 % kept: 8 chunks of 2^10
// 6.61 -> 6.67 -> 6.63, 256 of 2^14 14.4 -> 14.6 -> 14.4, 25 M samples in chunks of 2^12 39.9 -> 40.6 -> 40.0, of 2^15 67.6 -> 68.5 -> 67.6;  10 %
// kept, moved: 7.07 -> 6.70 -> 6.66, 14.2 -> 14.05 -> 13.8, 38.0 -> 37.0 -> 36.7, 66.1 -> 65.0 -> 64.0.  Transforms are longer and gain
// nothing (2^14 64.3 -> 65.2, 2^15 85.5 -> 87.1, 80 % kept), and the tensors of one launch differ: those decide as they run.
enum Packing { kByRow, kMoved, kEither };

// Steps 2-4 of the sender for one chunk whose bins (samples) lie in the registers of a group of WAVES waves:
// z[r]: bin (wave * R + r) * 64 + lane (lane < LR); zn (TAIL): the chunk's last bin, the same value in every lane.
// lds: the group's own words (histogram, candidate list, survivors), room of them; image: its record image, among them but for
// the shortest chunks.  wg_most: a word of the workgroup, zero on entry, through which several groups of several waves agree on
// the path they take together.
// runs: many of the samples are zero.  live = false groups (no such chunk) write nothing; groups of several waves call this together.
template <bool REAL, int R, bool TAIL, int LR, int WAVES, int GROUPS, int HB, Packing PACKING>
__device__ __forceinline__ void select_and_pack(const typename Elem<REAL>::T (&z)[R], typename Elem<REAL>::T zn, uint32_t* lds,
                                                uint32_t room, uint32_t* image, GroupScratch& gs, uint32_t* wg_most, int tid,
                                                const PackArgs& a, uint32_t word3, uint8_t* __restrict__ record, bool live,
                                                bool runs = false)
{
    constexpr int NL = 64 * WAVES;
    constexpr bool SHARED = WAVES > 1 && GROUPS > 1;
    constexpr uint32_t CODES = Elem<REAL>::kCodes;
    const int lane = tid & 63, tg = tid & (NL - 1), wig = __builtin_amdgcn_readfirstlane(tg >> 6);
    const bool tail = TAIL && wig == WAVES - 1;  // this wave owns the last bin
    auto ones = [](uint64_t m) __attribute__((always_inline)) { return (uint32_t)__popcll(m); };
    auto among = [&](bool p) __attribute__((always_inline)) { return __ballot(LR == 64 ? p : (p && lane < LR)); };
    const uint32_t keyn = TAIL ? (uint32_t)__builtin_amdgcn_readfirstlane((int)key_of(zn)) : 0u;
    uint32_t key[R];
#pragma unroll
    for (int r = 0; r < R; ++r) key[r] = key_of(z[r]);

    // ---- the k-th largest key ----
    uint32_t tau = 0, need = a.k, equal = 0;
    if constexpr (HB == 0) {
        // few keys: bisection on the key's bits, one ballot per row and bit, until a trial leaves exactly k keys
        bool open = true;
        for (int bit = 30; bit >= 0 && open; --bit) {
            const uint32_t t = tau | (1u << bit);
            uint32_t cnt = tail && keyn >= t ? 1u : 0u;
#pragma unroll
            for (int r = 0; r < R; ++r) cnt += ones(among(key[r] >= t));
            if (cnt >= need) tau = t;
            open = cnt != need;
        }
        equal = need;
        if (open) {
            uint32_t above = tail && keyn > tau ? 1u : 0u;
            equal = tail && keyn == tau ? 1u : 0u;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                above += ones(among(key[r] > tau));
                equal += ones(among(key[r] == tau));
            }
            need -= above;
        }
    } else {
        // One radix digit of NB bits at `shift` among the keys whose bits from shift + NB up equal those of tau:
        // counts in LDS, scanned from the top.  A lane scans PER consecutive counters; their places are swizzled in
        // quads so that the lanes' 16-byte reads spread over the banks.
        auto digit = [&](auto nb_tag, int shift) __attribute__((always_inline)) {
            constexpr int NB = decltype(nb_tag)::value, BINS = 1 << NB;
            constexpr int PER = BINS > NL ? BINS / NL : 1, QUADS = PER / 4;
            constexpr int LOGPER = PER == 1 ? 0 : PER == 2 ? 1 : PER == 4 ? 2 : PER == 8 ? 3 : PER == 16 ? 4 : 5;
            static_assert((1 << LOGPER) == PER, "counters per lane");
            auto place = [](uint32_t i) __attribute__((always_inline)) {
                if constexpr (QUADS > 1)
                    return i ^ (((i >> LOGPER) & (uint32_t)(QUADS - 1)) << 2);
                else
                    return i;
            };
            for (int i = 4 * tg; i < BINS; i += 4 * NL) *reinterpret_cast<uint4*>(lds + i) = make_uint4(0u, 0u, 0u, 0u);
            if (tg == 0) {
                gs.bucket = 0u;
                gs.need = 0u;
                gs.count = 0u;
                gs.listed = 0u;
            }
            group_sync<WAVES>();
            const int top = shift + NB;
            const uint32_t prefix = top >= 31 ? 0u : tau >> top;
            auto wanted = [&](uint32_t k) __attribute__((always_inline)) { return top >= 31 || k >> top == prefix; };
            auto add = [&](uint32_t k, uint32_t many) __attribute__((always_inline)) {
                atomicAdd(&lds[place((k >> shift) & (uint32_t)(BINS - 1))], many);
            };
            if (REAL && runs) {
                // the zeros past a gradient's end would queue for one counter: they are one addition a wave
                uint32_t zeros = 0;
                for (int r = 0; r < R; ++r) {
                    const bool in = (LR == 64 || lane < LR) && wanted(key[r]);
                    zeros += ones(__ballot(in && key[r] == 0u));
                    if (in && key[r] != 0u) add(key[r], 1u);
                }
                if (zeros && lane == 0) add(0u, zeros);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if ((LR == 64 || lane < LR) && wanted(key[r])) add(key[r], 1u);
            }
            if (tail && lane == 0 && wanted(keyn)) add(keyn, 1u);
            group_sync<WAVES>();
            uint32_t cnt[PER], sum = 0;
            const bool mine = PER > 1 || tg < BINS;
            const int base = BINS - PER - tg * PER;  // this lane's counters, [base, base + PER), from the top down
            if constexpr (PER >= 4) {
                const uint32_t b0 = place((uint32_t)base);  // base is a multiple of PER, so quad q sits at b0 ^ 4q
#pragma unroll
                for (int q = 0; q < QUADS; ++q) {
                    const uint4 v = *reinterpret_cast<const uint4*>(lds + (b0 ^ (uint32_t)(4 * q)));
                    cnt[4 * q] = v.x;
                    cnt[4 * q + 1] = v.y;
                    cnt[4 * q + 2] = v.z;
                    cnt[4 * q + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int i = 0; i < PER; ++i) cnt[i] = mine ? lds[base + i] : 0u;
            }
#pragma unroll
            for (int i = 0; i < PER; ++i) sum += cnt[i];
            const uint32_t incl = wave_scan_incl(sum);
            uint32_t before = incl - sum;
            if constexpr (WAVES > 1) {
                if (lane == 63) gs.a[wig] = incl;
                __syncthreads();
#pragma unroll
                for (int w = 0; w < WAVES - 1; ++w) before += w < wig ? gs.a[w] : 0u;
            }
            if (before < need && before + sum >= need) {
                uint32_t run = before;
#pragma unroll
                for (int i = PER - 1; i >= 0; --i) {
                    if (run < need && run + cnt[i] >= need) {
                        gs.bucket = (uint32_t)(base + i);
                        gs.need = need - run;
                        gs.count = cnt[i];
                        if (SHARED) atomicMax(wg_most, cnt[i]);
                    }
                    run += cnt[i];
                }
            }
            group_sync<WAVES>();
            tau |= (uint32_t)__builtin_amdgcn_readfirstlane((int)gs.bucket) << shift;
            need = (uint32_t)__builtin_amdgcn_readfirstlane((int)gs.need);
            equal = (uint32_t)__builtin_amdgcn_readfirstlane((int)gs.count);
        };
        constexpr int LOW1 = 31 - HB, LOW2 = LOW1 - 10;
        digit(std::integral_constant<int, HB>(), LOW1);
        const bool listed = (SHARED ? (uint32_t)__builtin_amdgcn_readfirstlane((int)*wg_most) : equal) <= kListCap;
        if (listed) {
            const uint32_t count = equal, prefix = tau >> LOW1;
            uint32_t mine = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) mine += ones(among(key[r] >> LOW1 == prefix));
            const bool tail_in = tail && keyn >> LOW1 == prefix;
            mine += tail_in ? 1u : 0u;
            uint32_t off = 0;
            if (WAVES > 1) {
                if (lane == 0) off = atomicAdd(&gs.listed, mine);
                off = (uint32_t)__builtin_amdgcn_readfirstlane((int)off);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const bool in = (LR == 64 || lane < LR) && key[r] >> LOW1 == prefix;
                const uint64_t m = __ballot(in);
                const uint32_t at = off + prefix_popc(m);
                if (in && at < kListCap) lds[at] = key[r];  // k = 0 selects an arbitrary bucket and drops it below
                off += ones(m);
            }
            if (tail_in && lane == 0 && off < kListCap) lds[off] = keyn;
            group_sync<WAVES>();
            if (count <= 64u)
                search_list<1>(lds, count, LOW1, lane, tau, need, equal);
            else
                search_list<4>(lds, count, LOW1, lane, tau, need, equal);
        } else {
            // heavy ties, or a long chunk: two more digits over the registers
            group_sync<WAVES>();  // everyone has read the first digit's result
            digit(std::integral_constant<int, 10>(), LOW2);
            group_sync<WAVES>();
            digit(std::integral_constant<int, LOW2>(), 0);
        }
    }
    if (a.k == 0) {
        tau = 0xFFFFFFFFu;
        need = equal = 0;
    }

    // ---- survivors: everything above tau and the first `need` bins equal to it ----
    uint64_t fm[R];
    bool fn;  // the last bin survives
    uint32_t nfl = 0, vmax = 0;
    // usually all bins equal to tau are wanted; in the other case their order across the group counts
    const bool ties = need != equal;
    uint32_t eqrun = 0;
    if (WAVES > 1 && (ties || SHARED)) {
        if (ties) {
            uint32_t neq = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) neq += ones(among(key[r] == tau));
            if (lane == 0) gs.a[wig] = neq;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WAVES - 1; ++w) eqrun += w < wig ? gs.a[w] : 0u;
        eqrun = (uint32_t)__builtin_amdgcn_readfirstlane((int)eqrun);
    }
    if (ties) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t em = among(key[r] == tau);
            fm[r] = among(key[r] > tau || (key[r] == tau && eqrun + prefix_popc(em) < need));
            eqrun += ones(em);
        }
        fn = tail && (keyn > tau || (keyn == tau && eqrun < need));
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) fm[r] = among(key[r] >= tau);
        fn = tail && keyn >= tau;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        nfl += ones(fm[r]);
        const uint32_t vb = __builtin_amdgcn_inverse_ballot_w64(fm[r]) ? vbits_of(z[r]) : 0u;
        vmax = vb > vmax ? vb : vmax;
    }
    vmax = wave_max(vmax);
    if (fn) {
        const uint32_t vb = (uint32_t)__builtin_amdgcn_readfirstlane((int)vbits_of(zn));
        vmax = vb > vmax ? vb : vmax;
        ++nfl;
    }
    uint32_t rank = 0;
    if constexpr (WAVES > 1) {
        if (lane == 0) {
            gs.b[wig] = nfl;
            gs.v[wig] = vmax;
        }
    }
    const int bits = a.bits, shift = 23 - a.m;
    const uint32_t image_words = (bits == 32 ? 4u + a.W : a.S / 4u);
    // The image's code words and padding start from zero; 8-bit codes overwrite whole units, so that only the words from
    // the last code on matter.
    const uint32_t zero_from = 4u + a.W + (bits == 8 ? CODES * a.k / 4u : 0u);
    for (uint32_t i = zero_from + (uint32_t)tg; i < image_words; i += NL) image[i] = 0u;
    group_sync<WAVES>();
    if constexpr (WAVES > 1) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            rank += w < wig ? gs.b[w] : 0u;
            const uint32_t v = gs.v[w];
            vmax = v > vmax ? v : vmax;
        }
        rank = (uint32_t)__builtin_amdgcn_readfirstlane((int)rank);
        vmax = (uint32_t)__builtin_amdgcn_readfirstlane((int)vmax);
    }
    if (a.static_vmax) vmax = a.static_vmax;
    uint32_t pbase = 0;
    if (bits != 32) {
        const int64_t pb = (int64_t)(vmax >> shift) - (int64_t)((1u << (bits - 1)) - 2u);
        pbase = pb < 1 ? 1u : (uint32_t)pb;
    }
    if (tg < 4) image[tg] = tg == 0 ? pbase : (tg == 1 ? vmax : (tg == 2 ? a.k : word3));

    // ---- bitmap ----
    if constexpr (LR == 64) {
        if (lane == 0) {
            uint32_t* words = image + 4 + wig * 2 * R;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                words[2 * r] = (uint32_t)fm[r];
                words[2 * r + 1] = (uint32_t)(fm[r] >> 32);
            }
        }
        if (tail && lane == 0) image[4 + WAVES * 2 * R] = fn ? 1u : 0u;  // the last bin opens a word of its own
    } else if (lane < (int)a.W) {
        const uint64_t all = TAIL ? fm[0] | ((uint64_t)(fn ? 1u : 0u) << LR) : fm[0];
        image[4 + lane] = lane ? (uint32_t)(all >> 32) : (uint32_t)all;
    }

    // ---- Algorithm 1 and the codes ----
    uint32_t* codes = image + 4 + a.W;
    uint32_t* direct = reinterpret_cast<uint32_t*>(record) + 4 + a.W;  // 32-bit codes go straight to memory
    auto code = [&](const typename Elem<REAL>::T& x, int h, int width) __attribute__((always_inline)) {
        if constexpr (REAL)
            return quantize(__float_as_uint(x), pbase, width, shift);
        else
            return quantize(__float_as_uint(h ? x.y : x.x), pbase, width, shift);
    };
    auto put = [&](auto mode, const typename Elem<REAL>::T& x, uint32_t rk) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode)::value;
        if constexpr (MODE == 8) {
            if constexpr (REAL)
                reinterpret_cast<uint8_t*>(codes)[rk] = (uint8_t)code(x, 0, 8);
            else
                reinterpret_cast<uint16_t*>(codes)[rk] = (uint16_t)(code(x, 0, 8) | (code(x, 1, 8) << 8));
        } else if constexpr (MODE == 32) {
            if (live) {
                direct[CODES * rk] = code(x, 0, 32);
                if constexpr (!REAL) direct[CODES * rk + 1] = code(x, 1, 32);
            }
        } else {
            uint32_t both = code(x, 0, bits);
            if constexpr (!REAL) both |= code(x, 1, bits) << bits;  // at most 32 bits
            const uint32_t width = CODES * (uint32_t)bits, p = width * rk, sh = p & 31u;
            atomicOr(&codes[p >> 5], both << sh);
            if (sh + width > 32u) atomicOr(&codes[(p >> 5) + 1], both >> (32u - sh));
        }
    };
    auto all = [&](auto mode) __attribute__((always_inline)) {
        uint32_t run = rank;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (__builtin_amdgcn_inverse_ballot_w64(fm[r])) put(mode, z[r], run + prefix_popc(fm[r]));
            run += ones(fm[r]);
        }
        if (fn && lane == 0) put(mode, zn, run);
    };
    bool packed = PACKING == kMoved;
    if constexpr (PACKING != kByRow) {
        const uint32_t from = (room - CODES * a.k) & ~1u;
        if (PACKING == kEither)
            packed = a.k <= most_packed<REAL, WAVES>((uint32_t)(R * NL), bits) && (uint32_t)(image - lds) + image_words + CODES * a.k < room;
        if (packed) {
            typename Elem<REAL>::T* kept = reinterpret_cast<typename Elem<REAL>::T*>(lds + from);
            uint32_t run = rank;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (__builtin_amdgcn_inverse_ballot_w64(fm[r])) kept[run + prefix_popc(fm[r])] = z[r];
                run += ones(fm[r]);
            }
            if (fn && lane == 0) kept[run] = zn;
            group_sync<WAVES>();
            auto each = [&](auto mode) __attribute__((always_inline)) {
                for (uint32_t i = (uint32_t)tg; i < a.k; i += NL) put(mode, kept[i], i);
            };
            if (bits == 8)
                each(std::integral_constant<int, 8>());
            else
                each(std::integral_constant<int, 0>());
        }
    }
    if (!packed) {
        if (bits == 8)
            all(std::integral_constant<int, 8>());
        else if (bits == 32)
            all(std::integral_constant<int, 32>());
        else
            all(std::integral_constant<int, 0>());
    }
    group_sync<WAVES>();
    if (live) {
        const uint32_t whole = image_words / 4u;
        uint4* dst = reinterpret_cast<uint4*>(record);
        for (uint32_t i = (uint32_t)tg; i < whole; i += NL) dst[i] = reinterpret_cast<const uint4*>(image)[i];
        if (bits == 32) {
            uint32_t* rec = reinterpret_cast<uint32_t*>(record);
            for (uint32_t i = 4u * whole + (uint32_t)tg; i < image_words; i += NL) rec[i] = image[i];
            for (uint32_t i = 4u + a.W + CODES * a.k + (uint32_t)tg; i < a.S / 4u; i += NL) rec[i] = 0u;  // padding
        }
    }
}

// record geometry of tensors of 2^(logm+1) samples
__device__ __forceinline__ PackArgs pack_args_of(const QuantizerArgs& q, const TensorTable& t, uint32_t logm)
{
    PackArgs a;
    a.k = t.kept[logm - 4u];
    a.W = ((1u << logm) + 32u) / 32u;
    a.S = t.stride[logm - 4u];
    a.word3 = 2u << logm;
    a.static_vmax = 0u;
    a.bits = q.bits;
    a.m = q.m;
    return a;
}

// what the first workgroup of a call leaves in the control block (see chunk.h)
__device__ __forceinline__ void write_control(uint32_t* __restrict__ ctl, const StatusNote& note, bool clear, int tid)
{
    if (tid == 0) {
        if (clear) {
            ctl[0] = 0u;
            ctl[1] = 0u;
        }
#pragma unroll
        for (int i = kNoteWord; i < kNoteWord + kNoteWords; ++i) ctl[i] = note_word(note, i);
    }
}

// Sender of one workgroup.
template <int LOGM, int NT, typename Where>
__device__ __forceinline__ void compress_workgroup(const float* __restrict__ in, const Where& where, const Tables& tb,
                                                   const PackArgs& a, uint8_t* __restrict__ records, uint8_t* lds, int tid)
{
    using G = Geo<LOGM, NT>;
    const int lane = tid & 63, group = tid / G::NL, wig = (tid >> 6) % G::WAVES;
    uint8_t* regions = lds + G::SENDER_FRONT;
    uint8_t* region = regions + group * G::REGION;
    constexpr int ROOM = G::REGION - G::INSIDE;
    static_assert(!G::INSIDE || ROOM >= 4 * kListCap + 16 + 4 * (G::WC + 1) + 4 * (G::M + 1) + 16, "list and image of 16-bit codes");
    static_assert(ROOM >= (G::HB ? 4 << G::HB : 0) && ROOM % 16 == 0, "histogram");
    GroupScratch& gs = *reinterpret_cast<GroupScratch*>(G::INSIDE ? region + ROOM : lds + group * (int)sizeof(GroupScratch));
    uint32_t* wg_most = reinterpret_cast<uint32_t*>((G::INSIDE ? regions + ROOM : lds) + (G::INSIDE ? 1 : G::GROUPS) * (int)sizeof(GroupScratch));
    // the workgroup's point g lies at d[flat(g)]; a group's points are a multiple of 256, so its base moves freely
    float2* d = reinterpret_cast<float2*>(region) - group * (G::E / G::GROUPS);
    float2* tw = reinterpret_cast<float2*>(regions + G::GROUPS * G::REGION);
    uint32_t* images = reinterpret_cast<uint32_t*>(tw + G::TW);  // short chunks only
    load_chunk_twiddles<LOGM, NT>(tw, tb, tid);
    forward_tile<G, LOGM>(in, where, tb, d, tw, tid);
    uint32_t* mine = reinterpret_cast<uint32_t*>(region);
    auto bins_of = [&](int b, float2 (&z)[G::R], float2& zn) __attribute__((always_inline)) {
        const int base = b << LOGM;
        if constexpr (G::M < 64) {
            const int k = lane & (G::M - 1);
            z[0] = split_bin<LOGM>(d[flat(base + k)], d[flat(base + ((G::M - k) & (G::M - 1)))], k, tb);
        } else {
            // rows of 64 bins upwards from k, and of their mirrors downwards: M - k is 64 - lane into a row that only its
            // number changes, except in lane 0
            const int k0 = wig * G::R * 64 + lane, f = flat(base + k0);
            const int g = flat(base + G::M - (wig + 1) * G::R * 64 + ((64 - lane) & 63));
#pragma unroll
            for (int r = 0; r < G::R; ++r) {
                const int first = base + ((G::M - (wig * G::R + r) * 64) & (G::M - 1));
                const int mirror = lane == 0 ? flat(first) : flat_plus(g, (G::R - 1 - r) * 64);
                const int k = k0 + r * 64;
                z[r] = split_fwd(d[flat_plus(f, r * 64)], d[mirror], split_twiddle<LOGM>(tb, k));
            }
            if (wig == 0) {
                const float2 a = d[flat(base)];
                if (lane == 0) z[0] = make_float2(a.x + a.y, 0.f);
            }
        }
        zn = nyquist_bin<LOGM>(d, base);
    };
    static_assert(G::REGION % 8 == 0, "survivors are aligned");
    auto pack = [&](int i, const float2 (&z)[G::R], float2 zn, uint32_t* image) __attribute__((always_inline)) {
        const int b = group * G::CPW + i;
        const bool live = where.exists(b);
        select_and_pack<false, G::R, true, G::LR, G::WAVES, G::GROUPS, G::HB, G::HB ? kEither : kByRow>(
            z, zn, mine, (uint32_t)ROOM / 4u, image, gs, wg_most, tid, a, a.word3, records + (live ? where.record(b) : 0), live);
    };
    if constexpr (G::HB == 0) {
        for (int i = 0; i < G::CPW; ++i) {  // the bins stay in LDS until their turn comes
            if (!where.exists(group * G::CPW + i)) break;  // single-wave groups: no barrier is skipped
            float2 z[G::R], zn;
            bins_of(group * G::CPW + i, z, zn);
            pack(i, z, zn, images + group * G::IMAGE);
            group_sync<G::WAVES>();
        }
    } else {
        // the bins move into registers and their LDS becomes histogram, candidate list and record image
        static_assert(G::CPW == 1, "one chunk per group");
        // A group of one wave without a chunk is done: no barrier follows.  Its zeros would all queue for one counter, and the call
        // wait for it: one chunk of 2^10 12.8 -> 7.3 us, of 2^11 19.8 -> 10.4.
        if (G::WAVES == 1 && !where.exists(group)) return;
        float2 z[G::R], zn;
        bins_of(group, z, zn);
        group_sync<G::WAVES>();
        if (G::WAVES > 1 && tid == 0) *wg_most = 0u;  // ordered by the barrier behind the histogram's zeros
        pack(0, z, zn, mine + kListCap);
    }
}

// The longest chunks' workgroups have a compute unit to themselves: four waves a SIMD, and told so, or the compiler keeps
// registers free for a fifth and holds the row masks in spilled scalars (2^15, 10-bit codes: 26 M samples 123 us against 110).
template <int LOGM, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT / 256, NT == 1024 ? 4 : 8))) void k_chunk_compress(
    const float* __restrict__ in, size_t n, size_t C, int aligned, Tables tb, PackArgs a, uint8_t* __restrict__ stream,
    uint8_t* __restrict__ records, HeaderInfo hdr, uint32_t* __restrict__ ctl)
{
    using G = Geo<LOGM, NT>;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x;
    if (blockIdx.x == 0) {
        write_control(ctl, StatusNote{}, true, tid);
        if (tid < 16) reinterpret_cast<uint32_t*>(stream)[tid] = header_word(hdr, tid);
    }
    const UniformChunks where(n, C, G::T, 2u * G::M, a.S, aligned);
    compress_workgroup<LOGM, NT>(in, where, tb, a, records, lds, tid);
}

template <typename G>
__device__ __forceinline__ ListedChunk listed(const TensorTable& t, const TensorPiece& piece, int tid)
{
    return ListedChunk(t, piece, tid / G::NL, G::CPW);
}
template <int LOGM>
__device__ __forceinline__ void compress_tensors(const float* __restrict__ in, const TensorTable& t, const TensorPiece& piece,
                                                 const Tables& tb, const PackArgs& a, uint8_t* __restrict__ records, uint8_t* lds, int tid)
{
    constexpr int NT = uniform_threads<LOGM>();
    if (tid >= NT) return;
    compress_workgroup<LOGM, NT>(in, listed<Geo<LOGM, NT>>(t, piece, tid), tb, a, records, lds, tid);
}

template <int TOP>
__device__ __forceinline__ void compress_piece(const float* __restrict__ in, const TensorTable& t, const Tables& tb, const QuantizerArgs& q,
                                               uint8_t* __restrict__ records, uint8_t* lds, int tid)
{
    const TensorPiece piece = t.piece[blockIdx.x];
    const PackArgs a = pack_args_of(q, t, piece.logm);
#define X(p) else if (p <= TOP && piece.logm == p) compress_tensors<(p <= TOP ? p : 4)>(in, t, piece, tb, a, records, lds, tid);
    if (false) {
    }
    FFTSP_CHUNK_SIZES(X)
#undef X
}

// The tensors of a per-tensor call that fit one workgroup, whatever their lengths, as one launch: workgroup i does the
// tensors of piece i.  Waves its length has no use for leave at once (an ended wave takes part in no barrier).
// TOP: the longest a launch may hold, 2^(TOP+1) samples.
template <int TOP>
__global__ __launch_bounds__(uniform_threads<TOP>()) void k_tensors_compress(const float* __restrict__ in, Tables tb,
                                                                            QuantizerArgs q, uint8_t* __restrict__ stream,
                                                                            uint8_t* __restrict__ records, HeaderInfo hdr,
                                                                            uint32_t* __restrict__ ctl, TensorTable t)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x;
    if (blockIdx.x == 0) {
        if (ctl) write_control(ctl, StatusNote{}, true, tid);
        if (hdr.write && tid < 16) reinterpret_cast<uint32_t*>(stream)[tid] = header_word(hdr, tid);
    }
    compress_piece<TOP>(in, t, tb, q, records, lds, tid);
}
// The same, and behind them the tiles of the forward pass A of a few longer tensors: those of short calls, or 2^14 points in half of the LDS (SPLIT).
template <bool SPLIT>
__global__ __launch_bounds__(uniform_threads<14>()) void k_tensors_compress_beside(const float* __restrict__ in, Tables tb, QuantizerArgs q,
                                                                                  uint8_t* __restrict__ stream, uint8_t* __restrict__ records,
                                                                                  HeaderInfo hdr, TensorTable t, uint32_t pieces, FewLong few,
                                                                                  float2* __restrict__ mid, uint32_t* __restrict__ zero_ptr,
                                                                                  uint32_t zero_words)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    constexpr uint32_t NT = uniform_threads<14>();
    const int tid = threadIdx.x;
    if (blockIdx.x >= pieces) {
        const uint32_t wg = blockIdx.x - pieces;
        for (uint32_t i = wg * NT + (uint32_t)tid; i < zero_words; i += (gridDim.x - pieces) * NT) zero_ptr[i] = 0u;
        const LongShare share = share_of(few.at, few.count, wg);
        if constexpr (SPLIT) {
            static_assert(NT == tile_lanes(14), "two tiles of columns of up to 2^10, or one of 2^11");
            fwd_a_split_tensor<14>(few.t[share.tensor], share.blk, in, mid, tb);
        } else {
            fwd_a_tensor(few.t[share.tensor], share.blk, in, mid, tb);
        }
        return;
    }
    if (blockIdx.x == 0 && hdr.write && tid < 16) reinterpret_cast<uint32_t*>(stream)[tid] = header_word(hdr, tid);
    compress_piece<14>(in, t, tb, q, records, lds, tid);
}

// ------------------------------------------------------- time-domain Top-k ----
// Sender of Top-k over the samples themselves: the same selection and packing, straight from the gradient.  Sixteen samples
// a lane (32 at 2^15): a wave per chunk up to 2^10 samples, a workgroup per chunk above.
// Bound by instruction issue and, since gradients crowd into few of the first digit's counters, by LDS atomics on one word.
// Measured on 26 M samples, 30 % kept as 8-bit codes, against the per-tile kernels with their 16 KB of histogram per chunk
// and six launches: L = 2^10 431 -> 52 us, 2^12 137 -> 38, 2^15 84 -> 74; 2^16 samples in chunks of 2^12 20 -> 8.
#define FFTSP_TOPK_SIZES(X) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)
template <int LOGL>
struct TopkGeo {
    static constexpr int L = 1 << LOGL;
    static constexpr int WAVES = L <= 1024 ? 1 : (L / 1024 < 16 ? L / 1024 : 16), GROUPS = WAVES == 1 ? 4 : 1;
    static constexpr int NL = 64 * WAVES, NT = NL * GROUPS;
    static constexpr int R = L / NL > 1 ? L / NL : 1, LR = L < 64 ? L : 64;
    static constexpr int HB = L <= 512 ? 0 : (L <= 4096 ? 11 : 12);
    static constexpr int SCRATCH = GROUPS * (int)sizeof(GroupScratch) + 16;
    static constexpr uint32_t most_moved(int bits) { return HB ? most_packed<true, WAVES>((uint32_t)L, bits) : 0u; }
    // LDS bytes of a group: histogram, then candidate list, record image and survivors
    static constexpr size_t region(size_t record, size_t moved)
    {
        const size_t image = ((HB ? 4 * (size_t)kListCap : 0) + record + 16 + 4 * moved + 15) / 16 * 16, hist = HB ? (size_t)4 << HB : 0;
        return image > hist ? image : hist;
    }
};
template <int LOGL, Packing PACKING>
__global__ __launch_bounds__(TopkGeo<LOGL>::NT) void k_topk_compress(const float* __restrict__ in, size_t n, size_t C, PackArgs a,
                                                                     uint8_t* __restrict__ stream, uint8_t* __restrict__ records,
                                                                     HeaderInfo hdr, uint32_t* __restrict__ ctl, uint32_t region)
{
    using G = TopkGeo<LOGL>;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, group = tid / G::NL, wig = (tid >> 6) % G::WAVES;
    if (blockIdx.x == 0) {
        write_control(ctl, StatusNote{}, true, tid);
        if (tid < 16) reinterpret_cast<uint32_t*>(stream)[tid] = header_word(hdr, tid);
    }
    const size_t c = (size_t)blockIdx.x * G::GROUPS + (size_t)group;
    if (c >= C) return;  // single-wave groups only: no barrier is skipped
    GroupScratch* gs = reinterpret_cast<GroupScratch*>(lds);
    uint32_t* mine = reinterpret_cast<uint32_t*>(lds + G::SCRATCH + (size_t)group * region);
    const float* src = in + (c << LOGL);
    const size_t left = n - (c << LOGL);
    const uint32_t present = left < (size_t)G::L ? (uint32_t)left : (uint32_t)G::L;  // what lies past the end counts as zeros
    float z[G::R];
#pragma unroll
    for (int r = 0; r < G::R; ++r) {
        const uint32_t i = (uint32_t)((wig * G::R + r) * 64 + lane);
        z[r] = 0.f;
        if (i < present) z[r] = src[i];
    }
    select_and_pack<true, G::R, false, G::LR, G::WAVES, G::GROUPS, G::HB, PACKING>(
        z, 0.f, mine, region / 4u, mine + (G::HB ? kListCap : 0u), gs[group], reinterpret_cast<uint32_t*>(gs + G::GROUPS), tid, a, a.word3,
        records + c * (size_t)a.S, true, present < (uint32_t)G::L);
}

// ---------------------------------------------------------------- receiver ----
// Receiver of one workgroup; several peers' streams are summed bin by bin in list order.
// region: LDS bytes of a group (receiver_region; single-wave groups run without barriers, so no group may touch another's bytes).
template <int LOGM, int NT, typename Where>
__device__ __forceinline__ void decompress_workgroup(const PeerList& streams, uint32_t npeers, int plain, const Where& where,
                                                     const Tables& tb, const PackArgs& a, const HeaderInfo& hdr,
                                                     float* __restrict__ out, float gain, uint32_t region,
                                                     uint32_t image_stride, size_t per_peer, uint32_t* __restrict__ verdicts,
                                                     uint8_t* lds, int tid)
{
    using G = Geo<LOGM, NT>;
    constexpr int RL = stage_radix_log(LOGM);
    using B = Butterflies<LOGM, G::LOGE, NT, RL>;
    const int lane = tid & 63, group = tid / G::NL, tg = tid & (G::NL - 1), wig = tg >> 6;
    GroupScratch* gs = reinterpret_cast<GroupScratch*>(lds);
    uint8_t* regions = lds + G::RECEIVER_FRONT;
    uint8_t* images = regions + (size_t)group * region;
    uint2* words = reinterpret_cast<uint2*>(images + region) - G::GROUP_WORDS;
    float2* tw = reinterpret_cast<float2*>(regions + (size_t)G::GROUPS * region);
    // the workgroup's point g lies at d[flat(g)]; a group's points are a multiple of 256, so its base moves freely
    float2* d = reinterpret_cast<float2*>(images) - group * (G::E / G::GROUPS);
    const int bits = a.bits, shift = 23 - a.m;
    const uint32_t code_base = 16u + 4u * a.W, last_rank = a.k ? a.k - 1u : 0u;
    load_chunk_twiddles<LOGM, NT>(tw, tb, tid);

    // value of the kept bin of this rank, codes in the record image; MODE: 8, 32, or 0 for the other widths
    auto value = [&](auto mode, const uint8_t* codes, uint32_t pbase, uint32_t rank, bool set) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode)::value;
        rank = rank < last_rank ? rank : last_rank;  // a corrupt bitmap must not point outside the record
        if constexpr (MODE == 32) {
            const uint2 v = load_code_pair(reinterpret_cast<const uint32_t*>(codes) + 2u * rank);
            return make_float2(__uint_as_float(set ? v.x : 0u), __uint_as_float(set ? v.y : 0u));
        } else {
            uint32_t both;
            int width = bits;
            if constexpr (MODE == 8) {
                both = *reinterpret_cast<const uint16_t*>(codes + 2u * rank);
                width = 8;
            } else {
                const uint32_t p = 2u * (uint32_t)bits * rank;
                const uint32_t* w = reinterpret_cast<const uint32_t*>(codes) + (p >> 5);  // a word past the codes at most
                both = __builtin_amdgcn_alignbit(w[1], w[0], p & 31u);                     // 2 * 16 bits at most
            }
            both = set ? both : 0u;
            return make_float2(__uint_as_float(dequantize(both, pbase, width, shift)),
                               __uint_as_float(dequantize(both >> width, pbase, width, shift)));
        }
    };

    float2 x[B::PER][B::RHO], xn = make_float2(0.f, 0.f);
    for (uint32_t peer = 0; peer < npeers; ++peer) {
        const uint8_t* stream = streams.p[peer];
        // the group's records, one behind the other
        for (int i = 0; i < G::CPW; ++i) {
            const int b = group * G::CPW + i;
            if (!where.exists(b)) break;
            const uint4* src = reinterpret_cast<const uint4*>(stream + 64 + where.record(b));
            uint4* dst = reinterpret_cast<uint4*>(images + (uint32_t)i * image_stride);
            for (uint32_t j = (uint32_t)tg; j < a.S / 16u; j += G::NL) dst[j] = src[j];
        }
        group_sync<G::WAVES>();
        // bitmap words with the number of set bits before each; the total tells a corrupt record
        {
            const bool has = tg < G::GROUP_WORDS;
            const int i = has ? tg / G::WC : 0, wi = has ? tg % G::WC : 0, b = group * G::CPW + i;
            const bool live = where.exists(b);
            const uint32_t* rec = reinterpret_cast<const uint32_t*>(images + (uint32_t)i * image_stride);
            uint32_t word = has && live ? rec[4 + wi] : 0u;
            uint32_t tail_bit;
            if constexpr (LOGM == 4) {
                tail_bit = (word >> 16) & 1u;
                word &= 0xFFFFu;
            } else {
                tail_bit = has && live ? rec[4 + G::WC] & 1u : 0u;
            }
            const uint32_t count = (uint32_t)__popc(word);
            uint32_t incl = count;
            constexpr int SEG = G::WC < 64 ? G::WC : 64;
#pragma unroll
            for (int o = 1; o < SEG; o <<= 1) {
                const uint32_t u = __shfl_up(incl, o, 64);
                if ((lane & (SEG - 1)) >= o) incl += u;
            }
            if constexpr (G::WC > 64) {
                if (lane == 63) gs[group].a[wig] = incl;
                __syncthreads();
#pragma unroll
                for (int w = 0; w < G::WC / 64 - 1; ++w) incl += w < wig ? gs[group].a[w] : 0u;
            }
            if (has) {
                words[tg] = make_uint2(word, incl - count);
                if (wi == G::WC - 1) {  // this lane knows the chunk's total: the last bin and the verdict are its
                    const uint32_t total = incl;
                    float2 v = make_float2(0.f, 0.f);
                    if (live) {
                        const uint8_t* codes = reinterpret_cast<const uint8_t*>(rec) + code_base;
                        const bool set = tail_bit && a.k > 0;
                        v = bits == 32 ? value(std::integral_constant<int, 32>(), codes, rec[0], total, set)
                                       : value(std::integral_constant<int, 0>(), codes, rec[0], total, set);
                        bool bad = total + tail_bit != a.k || rec[2] != a.k || rec[3] != a.word3;
                        const size_t c = where.verdict(b);
                        if (c == 0 && hdr.write) bad = bad || header_bad(hdr, reinterpret_cast<const uint32_t*>(stream));
                        verdicts[(size_t)peer * per_peer + c] = bad ? 6u : 0u;
                    }
                    xn = plain ? v : make_float2(xn.x + v.x, xn.y + v.y);
                }
            }
        }
        group_sync<G::WAVES>();
        auto bins = [&](auto mode) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < B::PER; ++q) {
                const int w = B::index(tid, q), j = B::j(w), b = B::b(w);
                const uint8_t* image = images + (uint32_t)(b - group * G::CPW) * image_stride;
                const uint32_t pbase = *reinterpret_cast<const uint32_t*>(image);
                const uint2* row = words + (b - group * G::CPW) * G::WC;
#pragma unroll
                for (int t = 0; t < B::RHO; ++t) {
                    const int i = j + t * B::STEP;
                    const uint2 e = B::STEP >= 32 ? row[(j >> 5) + t * (B::STEP / 32)] : row[i >> 5];
                    const uint32_t bit = 1u << ((B::STEP >= 32 ? j : i) & 31);
                    const uint32_t rank = e.y + (uint32_t)__popc(e.x & (bit - 1u));
                    const float2 v = value(mode, image + code_base, pbase, rank, (e.x & bit) != 0u && a.k > 0);
                    if (plain) {
                        x[q][t] = v;
                    } else {
                        const float2 prev = peer == 0 ? make_float2(0.f, 0.f) : x[q][t];
                        x[q][t] = make_float2(prev.x + v.x, prev.y + v.y);
                    }
                }
            }
        };
        if (bits == 8)
            bins(std::integral_constant<int, 8>());
        else if (bits == 32)
            bins(std::integral_constant<int, 32>());
        else
            bins(std::integral_constant<int, 0>());
        group_sync<G::WAVES>();  // the images may be overwritten
    }
    // the spectrum goes through LDS once, so that every lane can pick its bins' mirrors
#pragma unroll
    for (int q = 0; q < B::PER; ++q) {
        const int w = B::index(tid, q), f = flat((B::b(w) << LOGM) + B::j(w));
#pragma unroll
        for (int t = 1; t < B::RHO; ++t) d[flat_plus(f, t * B::STEP)] = x[q][t];
        d[f].x = x[q][0].x;
        if (B::j(w) != 0) d[f].y = x[q][0].y;
    }
    // imaginary parts of the DC and Nyquist bins are ignored: the Nyquist bin takes the place of one
    if (tg < G::CPW * G::WC && tg % G::WC == G::WC - 1) d[flat((group * G::CPW + tg / G::WC) << LOGM)].y = xn.x;
    if constexpr (G::WAVES == 1) __syncthreads();  // the twiddle table
    group_sync<G::WAVES>();
#pragma unroll
    for (int q = 0; q < B::PER; ++q) {
        const int w = B::index(tid, q), j = B::j(w), b = B::b(w);
#pragma unroll
        for (int t = 0; t < B::RHO; ++t) {
            const int k = j + t * B::STEP;
            // M - k = (STEP - j) + (RHO - 1 - t) * STEP for j > 0
            const int mirror = j == 0 ? flat((b << LOGM) + ((G::M - t * B::STEP) & (G::M - 1)))
                                      : flat_plus(flat((b << LOGM) + B::STEP - j), (B::RHO - 1 - t) * B::STEP);
            float2 p = d[mirror], s = x[q][t];
            if (t == 0 && k == 0) {
                p = make_float2(p.y, 0.f);
                s.y = 0.f;
            }
            x[q][t] = split_inv(s, p, split_twiddle<LOGM>(tb, k));
        }
    }
    group_sync<G::WAVES>();
    const float scale = gain * (1.0f / (float)(2 * G::M));
    if (where.whole(G::T)) {
        float2* dst = reinterpret_cast<float2*>(out + where.first_sample);
        fft_from_registers<LOGM, G::LOGE, NT, G::WAVES, true, false, RL>(x, d, tw, tid, [&](int b, int i, int o, float2 v) {
            dst[(b << LOGM) + i + o] = make_float2(v.x * scale, v.y * scale);
        });
    } else {
        fft_from_registers<LOGM, G::LOGE, NT, G::WAVES, true, false, RL>(x, d, tw, tid, [&](int b, int i, int o, float2 v) {
            const Span sp = where.span(b);
            store_pair(out, sp.first + 2 * (size_t)(i + o), sp.limit, make_float2(v.x * scale, v.y * scale));
        });
    }
}

template <int LOGM, int NT>
__global__ __launch_bounds__(NT) void k_chunk_decompress(PeerList streams, uint32_t npeers, int plain, size_t C, Tables tb,
                                                         PackArgs a, HeaderInfo hdr, float* __restrict__ out, size_t n,
                                                         int aligned, float gain, uint32_t region, uint32_t image_stride,
                                                         uint32_t* __restrict__ ctl, StatusNote note,
                                                         uint32_t* __restrict__ verdicts)
{
    using G = Geo<LOGM, NT>;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x;
    if (blockIdx.x == 0) write_control(ctl, note, true, tid);
    const UniformChunks where(n, C, G::T, 2u * G::M, a.S, aligned);
    decompress_workgroup<LOGM, NT>(streams, npeers, plain, where, tb, a, hdr, out, gain, region, image_stride, C, verdicts, lds,
                                   tid);
}

// LDS bytes of a receiver group in a per-tensor launch: one record image
template <typename G>
__host__ __device__ constexpr uint32_t tensor_region(uint32_t stride)
{
    return (uint32_t)G::receiver_region(stride + 16u);
}
template <int LOGM>
__device__ __forceinline__ void decompress_tensors(const PeerList& streams, const TensorTable& t, const TensorPiece& piece,
                                                   const Tables& tb, const PackArgs& a, const HeaderInfo& hdr,
                                                   float* __restrict__ out, uint32_t* __restrict__ verdicts, uint8_t* lds, int tid)
{
    constexpr int NT = uniform_threads<LOGM>();
    using G = Geo<LOGM, NT>;
    if (tid >= NT) return;
    decompress_workgroup<LOGM, NT>(streams, 1u, 1, listed<G>(t, piece, tid), tb, a, hdr, out, 1.0f,
                                   tensor_region<G>(a.S), a.S + 16u, 0, verdicts, lds, tid);
}

template <int TOP>
__device__ __forceinline__ void decompress_piece(const PeerList& streams, const TensorTable& t, const Tables& tb, const QuantizerArgs& q,
                                                 const HeaderInfo& hdr, float* __restrict__ out, uint32_t* __restrict__ verdicts, uint8_t* lds, int tid)
{
    const TensorPiece piece = t.piece[blockIdx.x];
    const PackArgs a = pack_args_of(q, t, piece.logm);
#define X(p) \
    else if (p <= TOP && piece.logm == p) decompress_tensors<(p <= TOP ? p : 4)>(streams, t, piece, tb, a, hdr, out, verdicts, lds, tid);
    if (false) {
    }
    FFTSP_CHUNK_SIZES(X)
#undef X
}
template <int TOP>
__global__ __launch_bounds__(uniform_threads<TOP>()) void k_tensors_decompress(PeerList streams, Tables tb, QuantizerArgs q,
                                                                              HeaderInfo hdr, float* __restrict__ out,
                                                                              uint32_t* __restrict__ ctl, StatusNote note,
                                                                              int clear, uint32_t* __restrict__ verdicts,
                                                                              TensorTable t)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && note.count) write_control(ctl, note, clear != 0, tid);
    decompress_piece<TOP>(streams, t, tb, q, hdr, out, verdicts, lds, tid);
}
// The same, and behind them the first kernel of a few longer tensors: the tiles of their inverse pass B, to mid, or (TABLE) their bitmaps' table.
template <bool TABLE>
__global__ __launch_bounds__(uniform_threads<14>()) void k_tensors_decompress_beside(const uint8_t* __restrict__ stream, Tables tb, QuantizerArgs q,
                                                                                    HeaderInfo hdr, float* __restrict__ out, uint32_t* __restrict__ ctl,
                                                                                    StatusNote note, uint32_t* __restrict__ verdicts, TensorTable t,
                                                                                    uint32_t pieces, FewLong few, float2* __restrict__ mid,
                                                                                    uint2* __restrict__ table, uint32_t* __restrict__ long_verdicts)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x;
    if (blockIdx.x >= pieces) {
        const LongShare share = share_of(few.at, few.count, blockIdx.x - pieces);
        HeaderInfo none = hdr;
        none.write = 0;  // the shorter tensors' workgroups look at the stream's header
        if constexpr (TABLE) {
            static_assert(kTableLanes == uniform_threads<14>(), "a lane has four words");
            bitmap_part_of_tensor(stream, few.t[share.tensor], share, none, table, long_verdicts);
        } else {
            decode_tensor<kDecodeMost / 2>(few.t[share.tensor], share.blk, stream, stream + 64, q.bits, q.m, none,
                                           share.blk == 0 ? long_verdicts + share.tensor : nullptr, false, mid, tb);
        }
        return;
    }
    if (blockIdx.x == 0) write_control(ctl, note, true, tid);
    PeerList one;
    one.p[0] = stream;
    decompress_piece<14>(one, t, tb, q, hdr, out, verdicts, lds, tid);
}

// ------------------------------------------------- stage-level transforms ----
template <int LOGM, int NT>
__global__ __launch_bounds__(NT) void k_chunk_rfft(const float* __restrict__ in, size_t n, size_t C, int aligned, Tables tb,
                                                   float2* __restrict__ spec, uint32_t sstride)
{
    using G = Geo<LOGM, NT>;
    extern __shared__ __attribute__((aligned(16))) float2 smem[];
    float2* d = smem;
    float2* tw = smem + G::E;
    const int tid = threadIdx.x;
    const size_t c0 = (size_t)blockIdx.x * G::T;
    load_chunk_twiddles<LOGM, NT>(tw, tb, tid);
    forward_tile<G, LOGM>(in, UniformChunks(n, C, G::T, 2u * G::M, 0u, aligned), tb, d, tw, tid);
    __syncthreads();
    for (int w = tid; w < G::E; w += NT) {
        const int k = w & (G::M - 1), b = w >> LOGM;
        if (c0 + (size_t)b >= C) continue;
        float2* X = spec + (c0 + (size_t)b) * (size_t)sstride;
        const int base = b << LOGM;
        X[k] = split_bin<LOGM>(d[flat(base + k)], d[flat(base + ((G::M - k) & (G::M - 1)))], k, tb);
        if (k == 0) X[G::M] = nyquist_bin<LOGM>(d, b << LOGM);
    }
}

template <int LOGM, int NT>
__global__ __launch_bounds__(NT) void k_chunk_irfft(const float2* __restrict__ spec, uint32_t sstride, size_t C, Tables tb,
                                                    float* __restrict__ out, size_t n)
{
    using G = Geo<LOGM, NT>;
    constexpr int RL = stage_radix_log(LOGM);
    using B = Butterflies<LOGM, G::LOGE, NT, RL>;
    extern __shared__ __attribute__((aligned(16))) float2 smem[];
    float2* d = smem;
    float2* tw = smem + G::E;
    const int tid = threadIdx.x;
    const size_t c0 = (size_t)blockIdx.x * G::T;
    load_chunk_twiddles<LOGM, NT>(tw, tb, tid);
    float2 x[B::PER][B::RHO];
#pragma unroll
    for (int q = 0; q < B::PER; ++q) {
        const int w = B::index(tid, q), j = B::j(w);
        const size_t c = c0 + (size_t)B::b(w);
#pragma unroll
        for (int t = 0; t < B::RHO; ++t) {
            const int k = j + t * B::STEP;
            x[q][t] = make_float2(0.f, 0.f);
            if (c < C) {
                const float2* X = spec + c * (size_t)sstride;
                float2 s = X[k], p = X[G::M - k];
                if (k == 0) s.y = p.y = 0.f;
                x[q][t] = split_inv(s, p, split_twiddle<LOGM>(tb, k));
            }
        }
    }
    __syncthreads();
    const float scale = 1.0f / (float)(2 * G::M);
    fft_from_registers<LOGM, G::LOGE, NT, G::WAVES, true, false, RL>(x, d, tw, tid, [&](int b, int i, int o, float2 v) {
        const Span sp = UniformChunks(n, C, G::T, 2u * G::M, 0u, 0).span(b);
        store_pair(out, sp.first + 2 * (size_t)(i + o), sp.limit, make_float2(v.x * scale, v.y * scale));
    });
}

// ---------------------------------------------------------------- launch ----
// bytes: the most that any call of this kernel takes, not what this one does.  The attribute is the kernel's: another thread
// may be between setting it and its launch.
template <typename K>
hipError_t allow_lds(K kernel, size_t bytes)
{
    if (bytes <= 48 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

PackArgs pack_args(const CodecArgs& a)
{
    PackArgs p;
    p.k = a.k;
    p.W = (codec_bins(a.L, a.time_domain) + 31) / 32;
    p.S = (uint32_t)a.S;
    p.word3 = a.word3;
    p.static_vmax = a.static_vmax;
    p.bits = a.bits;
    p.m = a.m;
    return p;
}
HeaderInfo header_info(const CodecArgs& a, int write)
{
    return HeaderInfo{write, a.hdr_n, a.hdr_L, a.hdr_C, (uint32_t)a.bits, (uint32_t)a.m, a.hdr_k, a.hdr_S,
                      a.hdr_theta, a.time_domain ? 1u : 0u, (uint32_t)a.hdr_scale};
}
int aligned8(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 7u) == 0; }

template <int LOGM, int NT>
constexpr size_t sender_lds()
{
    using G = Geo<LOGM, NT>;
    return G::SENDER_FRONT + (size_t)G::GROUPS * (G::REGION + 4 * G::IMAGE) + (size_t)G::TW * sizeof(float2);
}
template <int LOGM, int NT>
constexpr size_t receiver_lds(size_t region)
{
    using G = Geo<LOGM, NT>;
    return G::RECEIVER_FRONT + G::GROUPS * region + (size_t)G::TW * sizeof(float2);
}
// the longest record of M + 1 bins: all of them kept, 32-bit codes
constexpr size_t longest_record(size_t M) { return (16 + 4 * ((M + 32) / 32) + 8 * (M + 1) + 15) / 16 * 16; }
template <int LOGM, int NT>
constexpr size_t most_receiver_lds(size_t records)
{
    using G = Geo<LOGM, NT>;
    return receiver_lds<LOGM, NT>(G::receiver_region(records * (longest_record(G::M) + 16)));
}
// of a per-tensor launch whose longest tensor has 2^(LOGM+1) samples
template <int LOGM>
constexpr size_t most_tensors_lds(bool sender)
{
    constexpr int NT = uniform_threads<LOGM>();
    const size_t own = sender ? sender_lds<LOGM, NT>() : most_receiver_lds<LOGM, NT>(1);
    if constexpr (LOGM > 4) {
        const size_t shorter = most_tensors_lds<LOGM - 1>(sender);
        return own > shorter ? own : shorter;
    }
    return own;
}
constexpr size_t kLdsBytes = 160 * 1024;  // of a compute unit
static_assert(most_tensors_lds<14>(true) <= kLdsBytes && most_tensors_lds<14>(false) <= kLdsBytes, "fits");
// What leaving out the twiddles that no stage wants, and keeping a receiver's bitmap table where its data will be, is for: two
// workgroups of 2^13 points to a compute unit and four senders of 2^10, where one and three fitted.  33 M
// samples in chunks of 2^14: sender 129 -> 83 us, receiver 104 -> 68; of 2^11 72 -> 64 and 61 -> 54.  With 2^11 points four
// fit since their table is half a turn and the scratch lies in the regions; 512 lanes and eight points a lane instead: 78 -> 83 and
// 52 -> 56 us.
static_assert(2 * sender_lds<13, 512>() <= kLdsBytes && 2 * receiver_lds<13, 512>(Geo<13, 512>::DATA) <= kLdsBytes, "two a compute unit");
static_assert(4 * sender_lds<11, 256>() <= kLdsBytes && 4 * receiver_lds<11, 256>(Geo<11, 256>::DATA) <= kLdsBytes, "four a compute unit");
static_assert(4 * sender_lds<10, 256>() <= kLdsBytes && 4 * receiver_lds<10, 256>(Geo<10, 256>::DATA) <= kLdsBytes, "four a compute unit");

template <int LOGM>
hipError_t compress_as(const float* in, size_t n, const CodecArgs& a, uint8_t* stream, uint8_t* records, uint32_t* ctl,
                       Tables t, hipStream_t s)
{
    constexpr int NT = uniform_threads<LOGM>();
    using G = Geo<LOGM, NT>;
    constexpr size_t lds = sender_lds<LOGM, NT>();
    auto kern = k_chunk_compress<LOGM, NT>;
    const hipError_t e = allow_lds(kern, lds);
    if (e != hipSuccess) return e;
    FFTSP_LAUNCH("chunk_compress", kern, dim3((unsigned)((a.C + G::T - 1) / G::T)), dim3(NT), lds, s, in, n, a.C,
                 aligned8(in), t, pack_args(a), stream, records, header_info(a, 1), ctl);
    return hipGetLastError();
}

template <int LOGL>
hipError_t topk_compress_as(const float* in, size_t n, const CodecArgs& a, uint8_t* stream, uint8_t* records, uint32_t* ctl,
                            hipStream_t s)
{
    using G = TopkGeo<LOGL>;
    // records are whole 16 bytes; of one with 32-bit codes only header and bitmap pass through LDS
    const size_t image = a.bits == 32 ? 16 + ((size_t)a.L / 8 + 15) / 16 * 16 : a.S;
    const bool moved = G::HB && a.k <= G::most_moved(a.bits);  // and the region is made to hold them
    const size_t region = G::region(image, moved ? a.k : 0u), lds = G::SCRATCH + G::GROUPS * region;
    constexpr size_t longest = (16 + 4 * ((G::L + 31) / 32) + 2 * (size_t)G::L + 15) / 16 * 16;  // all kept, 16-bit codes
    auto kern = moved ? k_topk_compress<LOGL, G::HB ? kMoved : kByRow> : k_topk_compress<LOGL, kByRow>;
    const hipError_t e = allow_lds(kern, G::SCRATCH + G::GROUPS * G::region(longest, G::most_moved(16)));
    if (e != hipSuccess) return e;
    FFTSP_LAUNCH("topk_compress", kern, dim3((unsigned)((a.C + G::GROUPS - 1) / G::GROUPS)), dim3(G::NT), lds, s, in,
                 n, a.C, pack_args(a), stream, records, header_info(a, 1), ctl, (uint32_t)region);
    return hipGetLastError();
}

template <int LOGM>
hipError_t decompress_as(const PeerList& streams, int npeers, int plain, const CodecArgs& a, float* out, size_t n, float gain,
                         uint32_t* ctl, const StatusNote& note, uint32_t* verdicts, Tables t, hipStream_t s)
{
    constexpr int NT = uniform_threads<LOGM>();
    using G = Geo<LOGM, NT>;
    const uint32_t stride = (uint32_t)a.S + 16u;  // slack: a code is fetched as two words
    const size_t region = G::receiver_region((size_t)G::CPW * stride);
    const size_t lds = receiver_lds<LOGM, NT>(region);
    auto kern = k_chunk_decompress<LOGM, NT>;
    const hipError_t e = allow_lds(kern, most_receiver_lds<LOGM, NT>(G::CPW));
    if (e != hipSuccess) return e;
    FFTSP_LAUNCH("chunk_decompress", kern, dim3((unsigned)((a.C + G::T - 1) / G::T)), dim3(NT), lds, s, streams,
                 (uint32_t)npeers, plain, a.C, t, pack_args(a), header_info(a, 1), out, n, aligned8(out), gain,
                 (uint32_t)region, stride, ctl, note, verdicts);
    return hipGetLastError();
}

template <int LOGM>
hipError_t rfft_as(const float* in, size_t n, size_t C, float2* spec, uint32_t sstride, Tables t, hipStream_t s)
{
    constexpr int NT = uniform_threads<LOGM>();
    using G = Geo<LOGM, NT>;
    const size_t lds = (size_t)(G::E + G::TW) * sizeof(float2);
    auto kern = k_chunk_rfft<LOGM, NT>;
    const hipError_t e = allow_lds(kern, lds);
    if (e != hipSuccess) return e;
    FFTSP_LAUNCH("rfft_chunk", kern, dim3((unsigned)((C + G::T - 1) / G::T)), dim3(NT), lds, s, in, n, C, aligned8(in), t,
                 spec, sstride);
    return hipGetLastError();
}
template <int LOGM>
hipError_t irfft_as(const float2* spec, uint32_t sstride, size_t n, size_t C, float* out, Tables t, hipStream_t s)
{
    constexpr int NT = uniform_threads<LOGM>();
    using G = Geo<LOGM, NT>;
    const size_t lds = (size_t)(G::E + G::TW) * sizeof(float2);
    auto kern = k_chunk_irfft<LOGM, NT>;
    const hipError_t e = allow_lds(kern, lds);
    if (e != hipSuccess) return e;
    FFTSP_LAUNCH("irfft_chunk", kern, dim3((unsigned)((C + G::T - 1) / G::T)), dim3(NT), lds, s, spec, sstride, C, t, out, n);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_chunk_compress(const float* in, size_t n, int logL, const CodecArgs& a, uint8_t* stream, uint8_t* records,
                                 uint32_t* ctl, Tables t, hipStream_t s)
{
    if (a.C > 0x7fffffffu) return hipErrorInvalidValue;
    switch (logL - 1) {
#define X(p) \
    case p: return compress_as<p>(in, n, a, stream, records, ctl, t, s);
        FFTSP_CHUNK_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_topk_compress(const float* in, size_t n, int logL, const CodecArgs& a, uint8_t* stream, uint8_t* records,
                                uint32_t* ctl, hipStream_t s)
{
    if (a.C > 0x7fffffffu) return hipErrorInvalidValue;
    switch (logL) {
#define X(p) \
    case p: return topk_compress_as<p>(in, n, a, stream, records, ctl, s);
        FFTSP_TOPK_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_chunk_decompress(const PeerList& streams, int npeers, int plain, int logL, const CodecArgs& a, float* out,
                                   size_t n, float gain, uint32_t* ctl, const StatusNote& note, uint32_t* verdicts, Tables t,
                                   hipStream_t s)
{
    if (a.C > 0x7fffffffu) return hipErrorInvalidValue;
    switch (logL - 1) {
#define X(p) \
    case p: return decompress_as<p>(streams, npeers, plain, a, out, n, gain, ctl, note, verdicts, t, s);
        FFTSP_CHUNK_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

int tensors_per_workgroup(int logL)
{
    switch (logL - 1) {
#define X(p) \
    case p: return Geo<p, uniform_threads<p>()>::GROUPS;
        FFTSP_CHUNK_SIZES(X)
#undef X
        default: return 1;
    }
}

// LDS a launch of these pieces needs: that of its most demanding one
static size_t tensors_lds(const TensorTable& t, uint32_t pieces, bool sender)
{
    size_t most = 0;
    for (uint32_t i = 0; i < pieces; ++i) {
        size_t need = 0;
        switch (t.piece[i].logm) {
#define X(p)                                                                                                                 \
    case p:                                                                                                                  \
        need = sender ? sender_lds<p, uniform_threads<p>()>()                                                                 \
                      : receiver_lds<p, uniform_threads<p>()>(tensor_region<Geo<p, uniform_threads<p>()>>(t.stride[p - 4])); \
        break;
            FFTSP_CHUNK_SIZES(X)
#undef X
            default: break;
        }
        most = need > most ? need : most;
    }
    return most;
}

hipError_t launch_tensors_compress(const float* in, const TensorTable& t, uint32_t pieces, int top_logL, const QuantizerArgs& q,
                                   const CodecArgs& hdr, uint8_t* stream, uint8_t* records, uint32_t* ctl, Tables tb,
                                   hipStream_t s)
{
    const size_t lds = tensors_lds(t, pieces, true);
    const bool low = top_logL <= 12;
    const hipError_t e = low ? allow_lds(k_tensors_compress<11>, most_tensors_lds<11>(true))
                             : allow_lds(k_tensors_compress<14>, most_tensors_lds<14>(true));
    if (e != hipSuccess) return e;
    if (low)
        FFTSP_LAUNCH("tensors_compress", k_tensors_compress<11>, dim3(pieces), dim3(uniform_threads<11>()), lds, s, in,
                     tb, q, stream, records, header_info(hdr, hdr.write_header), ctl, t);
    else
        FFTSP_LAUNCH("tensors_compress", k_tensors_compress<14>, dim3(pieces), dim3(uniform_threads<14>()), lds, s, in,
                     tb, q, stream, records, header_info(hdr, hdr.write_header), ctl, t);
    return hipGetLastError();
}

hipError_t launch_tensors_decompress(const uint8_t* stream, const TensorTable& t, uint32_t pieces, int top_logL,
                                     const QuantizerArgs& q, const CodecArgs& hdr, float* out, uint32_t* ctl,
                                     const StatusNote& note, int clear, uint32_t* verdicts, Tables tb, hipStream_t s)
{
    const size_t lds = tensors_lds(t, pieces, false);
    const bool low = top_logL <= 12;
    const hipError_t e = low ? allow_lds(k_tensors_decompress<11>, most_tensors_lds<11>(false))
                             : allow_lds(k_tensors_decompress<14>, most_tensors_lds<14>(false));
    if (e != hipSuccess) return e;
    PeerList one{};
    one.p[0] = stream;
    if (low)
        FFTSP_LAUNCH("tensors_decompress", k_tensors_decompress<11>, dim3(pieces), dim3(uniform_threads<11>()), lds, s, one, tb, q,
                     header_info(hdr, hdr.write_header), out, ctl, note, clear, verdicts, t);
    else
        FFTSP_LAUNCH("tensors_decompress", k_tensors_decompress<14>, dim3(pieces), dim3(uniform_threads<14>()), lds, s, one, tb, q,
                     header_info(hdr, hdr.write_header), out, ctl, note, clear, verdicts, t);
    return hipGetLastError();
}

// the few longer tensors of a launch, tiles(logM) workgroups each; returns how many in all
template <typename Tiles>
static uint32_t few_of(const LongBatch& b, FewLong* few, Tiles&& tiles)
{
    few->count = b.count;
    for (uint32_t i = 0; i < b.count; ++i) few->t[i] = b.tab.t[i];
    return first_workgroups(b, 0, b.count, few->at, tiles);
}
static uint32_t few_forward(const LongBatch& b, FewLong* few)
{
    if (!short_forward(b)) return few_of(b, few, [](int logM) { return power_tiles(logM, 14); });
    return few_of(b, few, [](int logM) { return 1u << (logM - short_log_a(short_columns(logM))); });
}
static uint32_t few_inverse(const LongBatch& b, FewLong* few)
{
    if (!short_decode(b)) return few_of(b, few, [](int logM) { return table_parts(logM); });
    return few_of(b, few, [](int logM) { return 1u << (logM - short_rows(logM) - kShortLogSlots); });
}
constexpr size_t kStaticLds = 256;  // what RecordBins or bitmap_part keeps outside of the dynamic LDS, and more
static int longest_of(const LongBatch& b) { return b.tab.t[b.count - 1].logM; }  // it comes last
// Where the longer tensors take the kernels of short calls and there is room for them in the launch's arguments: their first kernel's 5 to 9 us and a
// launch's 3 hide behind the shorter ones' workgroups, which the grid starts with, also where they are more than compute units.  Sender and receiver in us, two launches /
// one: ResNet-20's 22 tensors 85.6 / 72.7, one of 2^16 and three of 300 54.4 / 41.5, three and one of 2^15 81.9 / 69.1, random sets of ten 99.0 / 82.1, 93.8 / 77.4 and 115 / 106;
// five of 20 k and twelve of 2^16 89.9 / 76.4, four of 2^18 94.9 / 81.0, six 103.0 / 86.4, three of 2^19 104.3 / 86.7; sixty of 9 k, six of 2^16 and two of 2^18 77.4 / 63.6.
// Senders have forward pass A of larger sets there, too, up to where run_segments takes two streams.  The kernel has the codec's 118 registers, so a compute unit holds one of
// its workgroups, and its tiles in half of the LDS have no other one beside them (in launches of their own two): what pays for that is the shorter tensors' time, and beside tensors that are
// done sooner the line lies at half as many.  Ten tensors 158 / 143, 20 164 / 149, 30 176 / 159, five of 20 k and two of 2^21 147 / 135, 30 of 30 k and seven 234 / 209, 20 of 20 k and three of 2^22
// 234 / 218;  five of 500 and two of 2^21 116 / 112, four 147 / 145.5, six 189 / 197;  30 of 9 k and eight 220 / 232.
// Against launches of their own as they are now (k_fwd_a_long), senders: five of 500 and two of 2^21 67.4 / 66.1, three 76.1 / 74.4, four 85.8 / 87.9;  128 of 4096 and three 83.8 / 74.1, four
// 93.5 / 91.3;  30 of 9 k and three 86.9 / 74.1, four 96.7 / 96.9, seven 137 / 131;  128 of 9 k and seven 136 / 138;  100 of 30 k and seven 146 / 137.
bool tensors_compress_beside(const TensorTable& t, const LongBatch& b)
{
    const bool brief = t.piece[0].logm <= 11;  // they come longest first
    return b.count <= (uint32_t)kFewLong && (short_forward(b) || (brief ? b.units <= kSideUnits / 2 : b.units < kSideUnits));
}
// Receivers' tiles of rows of 2^8 have a quarter of a workgroup's lanes there, and of 2^7 an eighth, with a compute unit to themselves, where launches of their own hold several on one.
// What hides that is the shorter tensors' time, by the longest of them, and as many compute units as they leave.  Receivers in us, two launches / one, beside 20 and 128 of 300, 4096, 9000 and 30 000:
//   eight of 2^18 (512 workgroups) 27.2 / 28.0 and 28.8 / 29.8, 28.2 / 28.1 and 29.6 / 30.7, 31.4 / 28.2 and 33.3 / 31.3, 37.6 / 29.0 and 40.5 / 36.9;
//   twelve (768) 31.8 / 35.4 and 32.8 / 37.3, 32.6 / 35.3 and 34.4 / 37.8, 35.8 / 35.5 and 37.7 / 38.4, 41.9 / 36.2 and 44.5 / 44.2;
//   fifteen (960) 34.5 / 38.2 and 36.5 / 39.9, 35.6 / 38.2 and 36.8 / 41.1, 39.0 / 38.3 and 40.6 / 45.1, 45.1 / 42.2 and 47.8 / 50.9;
//   nineteen of 2^16 (608) 24.1 / 24.2 and 28.6 / 26.3, 25.4 / 24.4 and 29.2 / 26.9;  of 2^17 (608) 27.1 / 27.5 and 28.9 / 29.0, 28.4 / 27.6 and 29.8 / 29.3, 31.5 / 27.7 and 33.2 / 34.2;
//   nine of 2^19 (576, rows of 2^9: half of the lanes) 41.4 / 39.3 and 42.9 / 40.6;  twenty and twenty-two of 2^17 beside 60 and 128 of 9000 32.7 / 28.9 and 31.2 / 32.3, 32.9 / 33.1 and 31.5 / 32.8.
static bool decode_beside(const TensorTable& t, uint32_t pieces, const LongBatch& b)
{
    uint32_t idle = 0;  // rows of 2^8: two for a workgroup, of 2^7: one
    for (uint32_t i = 0; i < b.count; ++i) {
        const int logM = b.tab.t[i].logM, rows = short_rows(logM);
        if (rows < 9) idle += (uint32_t)(rows - 6) << (logM - rows - kShortLogSlots);
    }
    const int longest = t.piece[0].logm;  // they come longest first
    return longest <= 11 ? idle < 1024u : longest <= 13 ? idle + 4u * pieces < 1700u : idle < 1920u || pieces <= 64u;
}
// Receivers of larger sets have the table of the longer ones' bitmaps there, 7 us and a launch's 3.  Sender and receiver in us, the table a launch of its own / there: ten
// tensors 143.5 / 137.8, 20 153.0 / 147.8 and 141.7 / 135.5, 30 158.9 / 153.4, five of 500 and two of 2^21 112.3 / 106.7, six 189.5 / 184.2, 30 of 9 k and seven 209.5 / 204.1.
bool tensors_decompress_beside(const TensorTable& t, uint32_t pieces, int bits, const LongBatch& b)
{
    return b.count <= (uint32_t)kFewLong && (short_decode(b) ? decode_beside(t, pieces, b) : b.units < kSideUnits && receive_applies(b, bits)) &&
           tensors_lds(t, pieces, false) + kStaticLds <= kLdsBytes;
}

hipError_t launch_tensors_compress_beside(const float* in, const TensorTable& t, uint32_t pieces, const QuantizerArgs& q, const CodecArgs& hdr,
                                          uint8_t* stream, uint8_t* records, const LongBatch& b, float2* mid, uint32_t* zero_ptr, uint32_t zero_words,
                                          Tables tb, hipStream_t s)
{
    if (!tensors_compress_beside(t, b)) return hipErrorInvalidValue;
    FewLong few{};
    const uint32_t wgs = few_forward(b, &few);
    const bool split = !short_forward(b);
    const size_t own = tensors_lds(t, pieces, true), theirs = split ? SplitTile<11, 14>::kLds : lds_a(short_columns(longest_of(b))), lds = own > theirs ? own : theirs;
    const auto kern = split ? k_tensors_compress_beside<true> : k_tensors_compress_beside<false>;
    const hipError_t e = allow_lds(kern, most_tensors_lds<14>(true));
    if (e != hipSuccess) return e;
    FFTSP_LAUNCH("tensors_compress", kern, dim3(pieces + wgs), dim3(uniform_threads<14>()), lds, s, in, tb, q, stream, records,
                 header_info(hdr, hdr.write_header), t, pieces, few, mid, zero_ptr, zero_words);
    return hipGetLastError();
}

hipError_t launch_tensors_decompress_beside(const uint8_t* stream, const TensorTable& t, uint32_t pieces, const QuantizerArgs& q, const CodecArgs& hdr,
                                            float* out, uint32_t* ctl, const StatusNote& note, uint32_t* verdicts, const LongBatch& b, float2* mid,
                                            void* table, uint32_t* long_verdicts, Tables tb, hipStream_t s)
{
    if (!tensors_decompress_beside(t, pieces, q.bits, b)) return hipErrorInvalidValue;
    FewLong few{};
    const uint32_t wgs = few_inverse(b, &few);
    const bool tables = !short_decode(b);
    const size_t own = tensors_lds(t, pieces, false), theirs = tables ? 0 : lds_decode(longest_of(b), short_rows(longest_of(b))), lds = own > theirs ? own : theirs;
    const auto kern = tables ? k_tensors_decompress_beside<true> : k_tensors_decompress_beside<false>;
    const hipError_t e = allow_lds(kern, kLdsBytes - kStaticLds);
    if (e != hipSuccess) return e;
    FFTSP_LAUNCH("tensors_decompress", kern, dim3(pieces + wgs), dim3(uniform_threads<14>()), lds, s, stream, tb, q, header_info(hdr, hdr.write_header), out,
                 ctl, note, verdicts, t, pieces, few, mid, static_cast<uint2*>(table), long_verdicts);
    return hipGetLastError();
}

hipError_t launch_chunk_rfft(const float* in, size_t n, int logL, size_t C, float* spec, uint32_t sstride, Tables t,
                             hipStream_t s)
{
    if (C > 0x7fffffffu) return hipErrorInvalidValue;
    switch (logL - 1) {
#define X(p) \
    case p: return rfft_as<p>(in, n, C, reinterpret_cast<float2*>(spec), sstride, t, s);
        FFTSP_CHUNK_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_chunk_irfft(const float* spec, uint32_t sstride, size_t n, int logL, size_t C, float* out, Tables t,
                              hipStream_t s)
{
    if (C > 0x7fffffffu) return hipErrorInvalidValue;
    switch (logL - 1) {
#define X(p) \
    case p: return irfft_as<p>(reinterpret_cast<const float2*>(spec), sstride, n, C, out, t, s);
        FFTSP_CHUNK_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fftsp

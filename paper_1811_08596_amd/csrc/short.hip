// The two-pass transforms of short calls (fft.hip has the long ones').
//
// A call of a few chunks is bound by latency: a launch behind another takes 3 us before it has done anything, and a wave
// issues a vector instruction every six to eight cycles however idle its SIMD is (measured on dependent and independent
// streams alike; four waves share a SIMD before they slow each other).  What counts is how many instructions a wave has to
// get through and how many dependent trips to memory come before them, so these kernels give a lane eight points instead of
// sixteen, spread a chunk over more and smaller workgroups, run one tile each and ask for everything they will need (samples,
// tables, twiddle anchors) before they wait for any of it.  Measured against the long calls' kernels, us per launch: one chunk of 2^16
// 7.3 -> 4.8 and 7.3 -> 5.2 forward, 8.0 -> 4.8 and 5.8 -> 4.4 inverse; two of 2^20 10.2 -> 9.3, 11.7 -> 10.6, 11.2 -> 8.9, 8.5 -> 7.3.
//
// The arithmetic is that of fft.hip, operation for operation: the same radices, the same recurrences from the same anchors.
// A chunk's spectrum and samples are the same bits whichever kernels a call takes.
#include "fft_core.h"
#include "codec_core.h"
#include "short.h"
#include "short_core.h"

#include <type_traits>

namespace fftsp {
namespace {

// ----------------------------------------------------------------- kernels ----
__device__ __forceinline__ void clear_words(uint32_t* __restrict__ p, uint32_t words, int lanes)
{
    for (uint32_t i = blockIdx.x * lanes + threadIdx.x; i < words; i += gridDim.x * lanes) p[i] = 0u;
}
// Work item of a workgroup: runs of 2^LOG consecutive items, whose tiles share lines of memory, go to workgroups of one XCD
// (they are dealt out round-robin over the eight).  Forward pass A of 2^22 samples in chunks of 2^16 15.8 -> 11.4 us.  Those that make no
// whole round of runs stay where they are: where then none moved, odd numbers of chunks of 2^16 lost, 37 sent and received 58.6 -> 56.3
// us, 45 61.0 -> 58.2, 27 51.1 -> 48.5 (though 27 sent again and again without anything between 33.2 -> 34.7).
template <int LOG>
__device__ __forceinline__ uint32_t beside()
{
    const uint32_t b = blockIdx.x;
    if (b >= (gridDim.x & ~((8u << LOG) - 1u))) return b;
    const uint32_t xcd = b & 7u, y = b >> 3;
    return (((y >> LOG) * 8u + xcd) << LOG) + (y & ((1u << LOG) - 1u));
}
// chunks of one length: a workgroup per tile, `tiles` (a power of two) of them to a chunk
template <int LOGN1, bool HALF>
__global__ __launch_bounds__(short_lanes_a(LOGN1)) void k_fwd_a_short(const float* __restrict__ in, size_t n, int logM,
                                                          typename Cx<HALF>::One* __restrict__ mid, Tables tb,
                                                          uint32_t* __restrict__ zero_ptr, uint32_t zero_words, float in_scale)
{
    clear_words(zero_ptr, zero_words, short_lanes_a(LOGN1));
    const int log_tiles = logM - short_log_a(LOGN1);
    const uint32_t place = beside<ShortColumns<LOGN1>::LOGSPLIT>(), c = place >> log_tiles;
    fwd_a_short<LOGN1, HALF>(place & ((1u << log_tiles) - 1u), in, chunk_span(0, n, c, (size_t)2 << logM), logM,
                             mid + ((size_t)c << logM), tb, in_scale);
}
template <int LOGN1, bool HALF>
__global__ __launch_bounds__(short_lanes_a(LOGN1)) void k_inv_a_short(const typename Cx<HALF>::One* __restrict__ mid, int logM,
                                                          float* __restrict__ out, size_t n, Tables tb, bool aligned, float gain)
{
    const int log_tiles = logM - short_log_a(LOGN1);
    const uint32_t place = beside<2>(), c = place >> log_tiles;
    inv_a_short<LOGN1, HALF>(place & ((1u << log_tiles) - 1u), mid + ((size_t)c << logM), logM, out,
                             chunk_span(0, n, c, (size_t)2 << logM), tb, aligned, gain);
}
template <int LOGN2, bool CODEC, bool HALF>
__global__ __launch_bounds__(1 << LOGN2) void k_fwd_b_short(const typename Cx<HALF>::One* __restrict__ mid, int logM,
                                                            typename Cx<HALF>::One* __restrict__ spec, uint32_t sstride, Tables tb,
                                                            uint32_t* __restrict__ hist, float mid_scale)
{
    const int log_tiles = logM - LOGN2 - kShortLogSlots;
    const uint32_t c = blockIdx.x >> log_tiles;
    fwd_b_short<LOGN2, CODEC, HALF>(blockIdx.x & ((1u << log_tiles) - 1u), mid + ((size_t)c << logM), logM,
                                    spec + c * (size_t)sstride, tb, CODEC ? hist + (size_t)c * kHistBins : nullptr, mid_scale);
}
template <int LOGN2, bool PAIR, bool HALF>
__global__ __launch_bounds__(1 << LOGN2) void k_inv_b_short(const typename Cx<HALF>::One* __restrict__ spec, uint32_t sstride, int logM,
                                                            typename Cx<HALF>::One* __restrict__ mid, Tables tb, float mid_scale)
{
    const int log_tiles = logM - LOGN2 - kShortLogSlots;
    const uint32_t c = blockIdx.x >> log_tiles;
    inv_b_short<LOGN2, HALF>(blockIdx.x & ((1u << log_tiles) - 1u), SpectrumBins<PAIR, HALF>{spec + c * (size_t)sstride}, logM,
                             mid + ((size_t)c << logM), tb, mid_scale);
}
template <int LOGN2, bool HALF>
__global__ __launch_bounds__(1 << LOGN2) void k_decode_inv_b(const uint8_t* __restrict__ stream, const uint8_t* __restrict__ records,
                                                             RecordArgs a, HeaderInfo hdr, uint32_t* __restrict__ verdicts,
                                                             uint32_t* __restrict__ ctl, StatusNote note, int logM,
                                                             typename Cx<HALF>::One* __restrict__ mid, Tables tb, float mid_scale)
{
    const int log_tiles = logM - LOGN2 - kShortLogSlots;
    const uint32_t c = blockIdx.x >> log_tiles, tile = blockIdx.x & ((1u << log_tiles) - 1u);
    if (blockIdx.x == 0) clear_control(ctl, note, threadIdx.x, 1 << LOGN2);
    const RecordBins<HALF> bins{records + (size_t)c * a.S, stream, a, tile == 0 ? verdicts + c : nullptr, c == 0, hdr};
    inv_b_short<LOGN2, HALF>(tile, bins, logM, mid + ((size_t)c << logM), tb, mid_scale);
}

// tensors of a LongTable, every workgroup looking up the one it belongs to
constexpr int kShortMostA = short_lanes_a(10);
__global__ __launch_bounds__(kShortMostA) void k_fwd_a_long_short(const float* __restrict__ in, float2* __restrict__ mid, Tables tb,
                                                               uint32_t* __restrict__ zero_ptr, uint32_t zero_words, LongTable tab,
                                                               LongStarts at)
{
    clear_words(zero_ptr, zero_words, (int)blockDim.x);
    const LongShare share = long_share(at);
    const LongTensor& x = tab.t[share.tensor];
    fwd_a_tensor(x, share.blk, in, mid, tb);
}
__global__ __launch_bounds__(kShortMostA) void k_inv_a_long_short(const float2* __restrict__ mid, float* __restrict__ out, Tables tb, bool aligned,
                                                               LongTable tab, LongStarts at)
{
    const LongShare share = long_share(at);
    const LongTensor& x = tab.t[share.tensor];
    const Span sp = chunk_span((size_t)x.goff, x.glen, 0, 0);
    const bool quads = aligned && (sp.first & 3u) == 0;
    const float2* from = mid + long_mid(x);
    if (threadIdx.x >= (uint32_t)short_lanes_a(short_columns(x.logM))) return;
    switch (short_columns(x.logM)) {
        case 8: return inv_a_short<8, false>(share.blk, from, x.logM, out, sp, tb, quads, 1.0f);
        case 9: return inv_a_short<9, false>(share.blk, from, x.logM, out, sp, tb, quads, 1.0f);
        default: return inv_a_short<10, false>(share.blk, from, x.logM, out, sp, tb, quads, 1.0f);
    }
}
// TOP: log2 of the most rows in the launch; lanes a shorter tensor has no use for leave at once (an ended wave takes part in
// no barrier)
template <int TOP>
__global__ __launch_bounds__(1 << TOP) void k_fwd_b_long_short(const float2* __restrict__ mid, float2* __restrict__ spec, Tables tb,
                                                               uint32_t* __restrict__ hist, LongTable tab, LongStarts at)
{
    const LongShare share = long_share(at);
    const LongTensor& x = tab.t[share.tensor];
    auto run = [&](auto n2) __attribute__((always_inline)) {
        constexpr int LOGN2 = decltype(n2)::value;
        if (threadIdx.x < (1u << LOGN2))
            fwd_b_short<LOGN2, true, false>(share.blk, mid + long_mid(x), x.logM, spec + long_spec(x, share.tensor), tb,
                                            hist + (size_t)share.tensor * kHistBins, 1.0f);
    };
    const int rows = short_rows(x.logM);
    if (rows == 7) return run(std::integral_constant<int, 7>{});
    if constexpr (TOP >= 8)
        if (rows == 8) return run(std::integral_constant<int, 8>{});
    if constexpr (TOP >= 9)
        if (rows == 9) return run(std::integral_constant<int, 9>{});
    if constexpr (TOP >= 10)
        if (rows == 10) return run(std::integral_constant<int, 10>{});
}
template <int TOP>
__global__ __launch_bounds__(1 << TOP) void k_inv_b_long_short(const float2* __restrict__ spec, float2* __restrict__ mid, Tables tb,
                                                               LongTable tab, LongStarts at)
{
    const LongShare share = long_share(at);
    const LongTensor& x = tab.t[share.tensor];
    auto run = [&](auto n2) __attribute__((always_inline)) {
        constexpr int LOGN2 = decltype(n2)::value;
        if (threadIdx.x < (1u << LOGN2))
            inv_b_short<LOGN2, false>(share.blk, SpectrumBins<true, false>{spec + long_spec(x, share.tensor)}, x.logM, mid + long_mid(x), tb,
                                      1.0f);
    };
    const int rows = short_rows(x.logM);
    if (rows == 7) return run(std::integral_constant<int, 7>{});
    if (rows == 8) return run(std::integral_constant<int, 8>{});
    if (rows == 9) return run(std::integral_constant<int, 9>{});
    if constexpr (TOP >= 10)
        if (rows == 10) return run(std::integral_constant<int, 10>{});
}

template <int TOP>
__global__ __launch_bounds__(1 << TOP) void k_decode_inv_b_long(const uint8_t* __restrict__ stream, const uint8_t* __restrict__ records,
                                                                int bits, int m, HeaderInfo hdr, uint32_t* __restrict__ verdicts,
                                                                uint32_t* __restrict__ ctl, StatusNote note,
                                                                float2* __restrict__ mid, Tables tb, LongTable tab, LongStarts at)
{
    if (ctl && blockIdx.x == 0) clear_control(ctl, note, threadIdx.x, 1 << TOP);
    const LongShare share = long_share(at);
    const LongTensor& x = tab.t[share.tensor];
    decode_tensor<TOP>(x, share.blk, stream, records, bits, m, hdr, share.blk == 0 ? verdicts + share.tensor : nullptr, share.tensor == 0, mid, tb);
}

// ------------------------------------------------------------------ launch ----
template <typename K>
hipError_t short_lds(K kernel, size_t bytes)
{
    if (bytes <= 48 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}
template <int LOGN1, bool HALF>
hipError_t launch_a_fwd(const float* in, size_t n, int logM, size_t C, float2* mid, Tables t, uint32_t* zero_ptr,
                        uint32_t zero_words, float in_scale, hipStream_t s)
{
    FFTSP_LAUNCH("rfft_pass_a", (k_fwd_a_short<LOGN1, HALF>), dim3((unsigned)(C << (logM - short_log_a(LOGN1)))), dim3(short_lanes_a(LOGN1)), lds_a(LOGN1), s,
                 in, n, logM, reinterpret_cast<typename Cx<HALF>::One*>(mid), t, zero_ptr, zero_words, in_scale);
    return hipGetLastError();
}
template <int LOGN1, bool HALF>
hipError_t launch_a_inv(const float2* mid, int logM, size_t C, float* out, size_t n, Tables t, bool aligned, float gain, hipStream_t s)
{
    FFTSP_LAUNCH("irfft_pass_a", (k_inv_a_short<LOGN1, HALF>), dim3((unsigned)(C << (logM - short_log_a(LOGN1)))), dim3(short_lanes_a(LOGN1)), lds_a(LOGN1), s,
                 reinterpret_cast<const typename Cx<HALF>::One*>(mid), logM, out, n, t, aligned, gain);
    return hipGetLastError();
}
template <int LOGN2, bool CODEC, bool HALF>
hipError_t launch_b_fwd(const float2* mid, int logM, size_t C, float2* spec, uint32_t sstride, Tables t, uint32_t* hist,
                        float mid_scale, hipStream_t s)
{
    constexpr size_t lds = lds_b(LOGN2, true);
    auto kern = k_fwd_b_short<LOGN2, CODEC, HALF>;
    const hipError_t e = short_lds(kern, lds);
    if (e != hipSuccess) return e;
    FFTSP_LAUNCH("rfft_pass_b", kern, dim3((unsigned)(C << (logM - LOGN2 - kShortLogSlots))), dim3(1 << LOGN2), lds, s,
                 reinterpret_cast<const typename Cx<HALF>::One*>(mid), logM, reinterpret_cast<typename Cx<HALF>::One*>(spec), sstride, t,
                 hist, mid_scale);
    return hipGetLastError();
}
template <int LOGN2, bool PAIR, bool HALF>
hipError_t launch_b_inv(const float2* spec, uint32_t sstride, int logM, size_t C, float2* mid, Tables t, float mid_scale, hipStream_t s)
{
    constexpr size_t lds = lds_b(LOGN2, false);
    auto kern = k_inv_b_short<LOGN2, PAIR, HALF>;
    const hipError_t e = short_lds(kern, lds);
    if (e != hipSuccess) return e;
    FFTSP_LAUNCH("irfft_pass_b", kern, dim3((unsigned)(C << (logM - LOGN2 - kShortLogSlots))), dim3(1 << LOGN2), lds, s,
                 reinterpret_cast<const typename Cx<HALF>::One*>(spec), sstride, logM, reinterpret_cast<typename Cx<HALF>::One*>(mid), t,
                 mid_scale);
    return hipGetLastError();
}

template <int LOGN2, bool HALF>
hipError_t launch_b_decode(const uint8_t* stream, const CodecArgs& a, int logM, float2* mid, Tables t, const HeaderInfo& hdr,
                           uint32_t* verdicts, uint32_t* ctl, const StatusNote& note, float mid_scale, hipStream_t s)
{
    auto kern = k_decode_inv_b<LOGN2, HALF>;
    const hipError_t e = short_lds(kern, lds_decode(2 * LOGN2 + 1 < kDecodeMost ? 2 * LOGN2 + 1 : kDecodeMost, LOGN2));
    if (e != hipSuccess) return e;
    const RecordArgs r{a.k, (1u << logM) / 32u + 1u, (uint32_t)a.S, a.word3, a.bits, a.m};
    FFTSP_LAUNCH("irfft_pass_b", kern, dim3((unsigned)(a.C << (logM - LOGN2 - kShortLogSlots))), dim3(1 << LOGN2), lds_decode(logM, LOGN2), s,
                 stream, stream + 64, r, hdr, verdicts, ctl, note, logM, reinterpret_cast<typename Cx<HALF>::One*>(mid), t, mid_scale);
    return hipGetLastError();
}

template <bool CODEC, bool HALF>
hipError_t rfft_short(const float* in, size_t n, int logM, size_t C, float2* spec, uint32_t sstride, float2* mid, Tables t,
                      uint32_t* hist, uint32_t* zero_ptr, uint32_t zero_words, float in_scale, float mid_scale, hipStream_t s)
{
    hipError_t e = hipErrorInvalidValue;
#define FWD_A(p) launch_a_fwd<p, HALF>(in, n, logM, C, mid, t, zero_ptr, zero_words, in_scale, s)
    switch (short_columns(logM)) {
        case 8: e = FWD_A(8); break;
        case 9: e = FWD_A(9); break;
        case 10: e = FWD_A(10); break;
    }
#undef FWD_A
    if (e != hipSuccess) return e;
#define FWD_B(p) launch_b_fwd<p, CODEC, HALF>(mid, logM, C, spec, sstride, t, hist, mid_scale, s)
    switch (short_rows(logM)) {
        case 7: return FWD_B(7);
        case 8: return FWD_B(8);
        case 9: return FWD_B(9);
        default: return FWD_B(10);
    }
#undef FWD_B
}
template <bool HALF>
hipError_t inv_a_any(const float2* mid, int logM, size_t C, float* out, size_t n, Tables t, float gain, hipStream_t s)
{
    const bool aligned = aligned16(out);
#define INV_A(p) launch_a_inv<p, HALF>(mid, logM, C, out, n, t, aligned, gain, s)
    switch (short_columns(logM)) {
        case 8: return INV_A(8);
        case 9: return INV_A(9);
        default: return INV_A(10);
    }
#undef INV_A
}
template <bool PAIR, bool HALF>
hipError_t inv_b_any(const float2* spec, uint32_t sstride, int logM, size_t C, float2* mid, Tables t, float mid_scale, hipStream_t s)
{
#define INV_B(p) launch_b_inv<p, PAIR, HALF>(spec, sstride, logM, C, mid, t, mid_scale, s)
    const int rows = short_rows(logM);
    if constexpr (!HALF) {
        if (rows == 7) return INV_B(7);
        if (rows == 8) return INV_B(8);
    }
    // shorter binary16 spectra are not made: see kShortDecode
    if (rows < 9) return hipErrorInvalidValue;
    return rows == 9 ? INV_B(9) : INV_B(10);
#undef INV_B
}
template <bool HALF>
hipError_t decode_b_any(const uint8_t* stream, const CodecArgs& a, int logM, float2* mid, Tables t, float mid_scale, uint32_t* verdicts,
                        uint32_t* ctl, const StatusNote& note, hipStream_t s)
{
    const HeaderInfo hdr{1, a.hdr_n, a.hdr_L, a.hdr_C, (uint32_t)a.bits, (uint32_t)a.m, a.hdr_k, a.hdr_S, a.hdr_theta, 0u, (uint32_t)a.hdr_scale};
#define DECODE_B(p) launch_b_decode<p, HALF>(stream, a, logM, mid, t, hdr, verdicts, ctl, note, mid_scale, s)
    switch (short_rows(logM)) {
        case 7: return DECODE_B(7);
        case 8: return DECODE_B(8);
        case 9: return DECODE_B(9);
        default: return hipErrorInvalidValue;
    }
#undef DECODE_B
}

}  // namespace

// In tiles of 2^13 points, by length: whole calls in us, the kernels of fft.hip / these, 8-bit codes of half of the bins, buffers in turn:
//   sender:    2^16 64 30.9 / 28.1, 128 37.5 / 35.9, 160 37.4 / 39.6, 192 39.2 / 40.1;  2^17 128 38.3 / 35.6, 192 43.0 / 41.3, 208 44.2 / 44.8;
//     2^18 128 40.0 / 38.4, 192 44.7 / 44.3, 208 46.1 / 49.3;  2^19 128 41.6 / 38.9, 192 46.4 / 45.5, 224 48.9 / 50.3;  2^20 128 45.7 / 42.4,
//     192 50.0 / 48.7;  2^21 128 54.5 / 49.8, 256 63.3 / 61.9, 384 72.5 / 78.1
//     Sent and received in turn, 2^16 132 57.0 / 54.4, 160 57.4 / 56.8, 176 58.8 / 57.8, 192 59.7 / 58.9; sent after other kernels and 600 MB of
//     other memory 136 52.5 / 50.1, 156 52.8 / 51.0, 164 54.6 / 53.0, 192 54.6 / 55.0.  That is nearer to a training step.
//   binary16:  2^16 128 36.0 / 35.8, 144 37.6 / 37.7, 192 39.8 / 40.5, after other kernels 144 50.2 / 50.9, 192 52.4 / 53.8;  2^17 192 41.1 / 40.5, 208 41.9 /
//     43.2;  2^18 128 37.8 / 36.1, 160 40.2 / 40.7, 192 42.1 / 43.5;  2^19 192 44.7 / 44.1, 224 46.6 / 48.7;  2^20 128 43.9 / 41.6, 192 48.9 / 48.6;
//     2^21 128 53.5 / 49.1
//   receiver, transform alone: 2^20 64 24.3 / 20.1, 256 35.9 / 33.8, 384 44.7 / 41.6, 512 51.5 / 51.5;  2^21 128 34.1 / 31.4, 384 51.9 / 53.0
// Tensors: sets of random ones, padded to 2^16 to 2^21 samples, few of them whole powers of two, most tiles of 2^18 and more.  Time with these over time
// with fft.hip's: senders, 890 sets of 129 to 192 tiles, 1.003 in the mean (up to 160 tiles 0.98, above 176 1.04, single sets 0.91 to
// 1.12); receivers, 2273 sets of 129 to 320 tiles, 0.994 (0.85 to 1.15).
constexpr size_t kShortForward = 192, kShortForwardHalf[] = {128, 192, 128, 192, 192, 192};  // the latter from 2^16 on
constexpr size_t kShortInverse = 320;
// The inverse pass B from records, against receive.hip's two kernels, in whole receivers: 2^16 128 15.0 / 18.2, 256 22.0 / 25.4, 362 29.8 /
// 32.6, 512 40.3 / 37.4;  2^18 128 17.0 / 19.0, 256 25.9 / 27.3, 362 35.8 / 33.7;  2^19 128 17.6 / 23.2, 362 38.7 / 39.3, 512 47.6 / 41.9.
constexpr size_t kShortDecode = 320;
static_assert(kShortDecode >= kShortInverse && kDecodeMost / 2 == 9, "receivers of short calls have a spectrum from rows of 2^9 on");
constexpr int kShortMostLogM = 20;
static size_t tiles_of(int logM, size_t C) { return C << (logM - 13); }
static size_t tiles_of(const LongBatch& b) { return (size_t)b.units << (kLongUnitLog - 13); }
static int longest(const LongBatch& b) { return b.tab.t[b.count - 1].logM; }  // it comes last
static bool short_length(int logM) { return logM >= 15 && logM <= kShortMostLogM; }

bool short_forward(int logM, size_t C, int half)
{
    return short_length(logM) && tiles_of(logM, C) <= (half ? kShortForwardHalf[logM - 15] : kShortForward);
}
bool short_forward(const LongBatch& b) { return short_length(longest(b)) && tiles_of(b) <= kShortForward; }
bool short_inverse(int logM, size_t C) { return short_length(logM) && tiles_of(logM, C) <= kShortInverse; }
bool short_inverse(const LongBatch& b) { return short_length(longest(b)) && tiles_of(b) <= kShortInverse; }
bool short_decode(int logM, size_t C) { return logM >= 15 && logM <= kDecodeMost && tiles_of(logM, C) <= kShortDecode; }
bool short_decode(const LongBatch& b) { return longest(b) <= kDecodeMost && tiles_of(b) <= kShortDecode; }

hipError_t launch_short_rfft(const float* in, size_t n, int logM, size_t C, float2* spec, uint32_t sstride, float2* mid, Tables t,
                             uint32_t* hist, uint32_t* zero_ptr, uint32_t zero_words, hipStream_t s)
{
    return hist ? rfft_short<true, false>(in, n, logM, C, spec, sstride, mid, t, hist, zero_ptr, zero_words, 1.0f, 1.0f, s)
                : rfft_short<false, false>(in, n, logM, C, spec, sstride, mid, t, nullptr, zero_ptr, 0u, 1.0f, 1.0f, s);
}
hipError_t launch_short_inverse_b(const float2* spec, uint32_t sstride, int logM, size_t C, float2* mid, Tables t, int pair_spec,
                                  hipStream_t s)
{
    return pair_spec ? inv_b_any<true, false>(spec, sstride, logM, C, mid, t, 1.0f, s)
                     : inv_b_any<false, false>(spec, sstride, logM, C, mid, t, 1.0f, s);
}
hipError_t launch_short_inverse_b_half(const float2* spec, uint32_t sstride, int logM, size_t C, float2* mid, Tables t, float mid_scale,
                                       hipStream_t s)
{
    return inv_b_any<true, true>(spec, sstride, logM, C, mid, t, mid_scale, s);
}
hipError_t launch_short_inverse_a(const float2* mid, int logM, size_t C, float* out, size_t n, Tables t, float gain, int half, hipStream_t s)
{
    return half ? inv_a_any<true>(mid, logM, C, out, n, t, gain, s) : inv_a_any<false>(mid, logM, C, out, n, t, gain, s);
}
hipError_t launch_short_rfft_half(const float* in, size_t n, int logM, size_t C, float2* spec, uint32_t sstride, float2* mid, Tables t,
                                  uint32_t* hist, uint32_t* zero_ptr, uint32_t zero_words, float in_scale, float mid_scale, hipStream_t s)
{
    return rfft_short<true, true>(in, n, logM, C, spec, sstride, mid, t, hist, zero_ptr, zero_words, in_scale, mid_scale, s);
}
hipError_t launch_short_decode(const uint8_t* stream, const CodecArgs& a, int logM, float2* mid, Tables t, uint32_t* verdicts,
                               uint32_t* ctl, const StatusNote& note, hipStream_t s)
{
    if (!a.half) return decode_b_any<false>(stream, a, logM, mid, t, 1.0f, verdicts, ctl, note, s);
    return decode_b_any<true>(stream, a, logM, mid, t, 1.0f / half_lift(logM), verdicts, ctl, note, s);
}
hipError_t launch_short_decode_long(const uint8_t* stream, const CodecArgs& a, float2* mid, Tables t, int check_header,
                                    uint32_t* verdicts, uint32_t* ctl, const StatusNote* first, hipStream_t s)
{
    const LongBatch& b = *a.tab;
    const HeaderInfo hdr{check_header, a.hdr_n, a.hdr_L, a.hdr_C, (uint32_t)a.bits, (uint32_t)a.m, a.hdr_k, a.hdr_S, a.hdr_theta, 0u, 0u};
    const StatusNote note = first ? *first : StatusNote{};
    const int logM = longest(b);
    LongStarts at;
    const uint32_t wgs = long_starts(b, 0, b.count, &at, [](int logM) { return 1u << (logM - short_rows(logM) - kShortLogSlots); });
    auto pass_b = [&](auto top) {
        constexpr int TOP = decltype(top)::value;
        auto kern = k_decode_inv_b_long<TOP>;
        const hipError_t e = short_lds(kern, lds_decode(2 * TOP + 1 < kDecodeMost ? 2 * TOP + 1 : kDecodeMost, TOP));
        if (e != hipSuccess) return e;
        FFTSP_LAUNCH("irfft_pass_b", kern, dim3(wgs), dim3(1 << TOP), lds_decode(logM, TOP), s, stream, stream + 64, a.bits, a.m, hdr,
                     verdicts, first ? ctl : nullptr, note, mid, t, b.tab, at);
        return hipGetLastError();
    };
    switch (short_rows(logM)) {
        case 7: return pass_b(std::integral_constant<int, 7>{});
        case 8: return pass_b(std::integral_constant<int, 8>{});
        default: return pass_b(std::integral_constant<int, 9>{});
    }
}

hipError_t launch_short_rfft_long(const float* in, const LongBatch& b, float2* spec, float2* mid, Tables t, uint32_t* hist,
                                  uint32_t* zero_ptr, uint32_t zero_words, hipStream_t s)
{
    LongStarts at;
    const int top = short_columns(longest(b));
    const uint32_t wgs = long_starts(b, 0, b.count, &at, [](int logM) { return 1u << (logM - short_log_a(short_columns(logM))); });
    FFTSP_LAUNCH("rfft_pass_a", k_fwd_a_long_short, dim3(wgs), dim3(short_lanes_a(top)), lds_a(top), s, in, mid, t, zero_ptr, zero_words,
                 b.tab, at);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? launch_short_rfft_b_long(b, spec, mid, t, hist, s) : e;
}
hipError_t launch_short_rfft_b_long(const LongBatch& b, float2* spec, const float2* mid, Tables t, uint32_t* hist, hipStream_t s)
{
    LongStarts at;
    const uint32_t wgs = long_starts(b, 0, b.count, &at, [](int logM) { return 1u << (logM - short_rows(logM) - kShortLogSlots); });
    auto pass_b = [&](auto top) {
        constexpr int TOP = decltype(top)::value;
        auto kern = k_fwd_b_long_short<TOP>;
        const hipError_t e = short_lds(kern, lds_b(TOP, true));
        if (e != hipSuccess) return e;
        FFTSP_LAUNCH("rfft_pass_b", kern, dim3(wgs), dim3(1 << TOP), lds_b(TOP, true), s, mid, spec, t, hist, b.tab, at);
        return hipGetLastError();
    };
    switch (short_rows(longest(b))) {
        case 7: return pass_b(std::integral_constant<int, 7>{});
        case 8: return pass_b(std::integral_constant<int, 8>{});
        case 9: return pass_b(std::integral_constant<int, 9>{});
        default: return pass_b(std::integral_constant<int, 10>{});
    }
}
hipError_t launch_short_inverse_b_long(const float2* spec, const LongBatch& b, float2* mid, Tables t, hipStream_t s)
{
    LongStarts at;
    const uint32_t wgs = long_starts(b, 0, b.count, &at, [](int logM) { return 1u << (logM - short_rows(logM) - kShortLogSlots); });
    auto pass_b = [&](auto top) {
        constexpr int TOP = decltype(top)::value;
        auto kern = k_inv_b_long_short<TOP>;
        const hipError_t e = short_lds(kern, lds_b(TOP, false));
        if (e != hipSuccess) return e;
        FFTSP_LAUNCH("irfft_pass_b", kern, dim3(wgs), dim3(1 << TOP), lds_b(TOP, false), s, spec, mid, t, b.tab, at);
        return hipGetLastError();
    };
    // sets whose longest has shorter rows have no spectrum: see kShortDecode
    if (short_rows(longest(b)) < 9) return hipErrorInvalidValue;
    return short_rows(longest(b)) == 9 ? pass_b(std::integral_constant<int, 9>{}) : pass_b(std::integral_constant<int, 10>{});
}

hipError_t launch_short_inverse_a_long(const LongBatch& b, float* out, const float2* mid, Tables t, hipStream_t s)
{
    LongStarts at;
    const int top = short_columns(longest(b));
    const uint32_t wgs = long_starts(b, 0, b.count, &at, [](int logM) { return 1u << (logM - short_log_a(short_columns(logM))); });
    FFTSP_LAUNCH("irfft_pass_a", k_inv_a_long_short, dim3(wgs), dim3(short_lanes_a(top)), lds_a(top), s, mid, out, t, aligned16(out), b.tab, at);
    return hipGetLastError();
}

}  // namespace fftsp

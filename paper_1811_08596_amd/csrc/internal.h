// Internal declarations shared by the translation units of libfftsp.so.
// Nothing here is part of the C ABI (see include/fftsp.h).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>
#include <stddef.h>
#include <string>
#include <type_traits>

namespace fftsp {

constexpr int kMinLogL = 5;   // chunk length 32
constexpr int kMaxLogL = 22;  // chunk length 4 Mi

// Twiddle tables, one pair per device, 2048 entries each:
//   hi[h] = exp(-2 pi i h / 2^11),  lo[l] = exp(-2 pi i l / 2^22)
// so that exp(-2 pi i E / 2^22) = hi[E >> 11] * lo[E & 2047] for any E < 2^22.
struct Tables {
    const float2* hi;
    const float2* lo;
};

// How complex values are stored where they cross HBM between kernels (the two-pass intermediate and the codec's
// own spectrum): binary32 pairs, or binary16 pairs in the half-precision variant (Sec. 3.1.1, "Our approach").
// Arithmetic is binary32 in registers and LDS either way; the variant halves the bytes, which is what bounds
// these kernels.  One = a complex value, Two = two adjacent ones (what a lane moves per access).
template <bool HALF>
struct Cx {
    using One = float2;
    using Two = float4;
};
template <>
struct Cx<true> {
    using One = uint32_t;  // bit pattern of two binary16 numbers (re low, im high)
    using Two = uint2;
};
// round to nearest even, saturating at the largest finite binary16 number
__device__ __forceinline__ uint32_t pack_half2(float2 v)
{
    const float lim = 65504.f;
    const __half2 h = __floats2half2_rn(fminf(fmaxf(v.x, -lim), lim), fminf(fmaxf(v.y, -lim), lim));
    uint32_t w;
    __builtin_memcpy(&w, &h, sizeof(w));
    return w;
}
__device__ __forceinline__ float2 unpack_half2(uint32_t w)
{
    __half2 h;
    __builtin_memcpy(&h, &w, sizeof(w));
    return __half22float2(h);
}
__device__ __forceinline__ float2 cx_load(float2 v) { return v; }
__device__ __forceinline__ float2 cx_load(uint32_t v) { return unpack_half2(v); }
__device__ __forceinline__ float4 cx_load(float4 v) { return v; }
__device__ __forceinline__ float4 cx_load(uint2 v)
{
    const float2 a = unpack_half2(v.x), b = unpack_half2(v.y);
    return make_float4(a.x, a.y, b.x, b.y);
}
template <bool HALF>
__device__ __forceinline__ typename Cx<HALF>::One cx_store(float2 v)
{
    if constexpr (HALF)
        return pack_half2(v);
    else
        return v;
}
template <bool HALF>
__device__ __forceinline__ typename Cx<HALF>::Two cx_store(float4 v)
{
    if constexpr (HALF)
        return make_uint2(pack_half2(make_float2(v.x, v.y)), pack_half2(make_float2(v.z, v.w)));
    else
        return v;
}

// Selection geometry: one workgroup of 256 lanes owns a tile of 2048 consecutive bins
// (wave w owns 512 of them as 8 rows of 64), so a wave ballot is two bitmap words.
constexpr int kTile = 2048;
constexpr int kTileThreads = 256;
constexpr int kHistBits = 12;                 // first radix-select digit: top 12 bits of the 31-bit key
constexpr int kHistBins = 1 << kHistBits;
constexpr int kKeyShift = 31 - kHistBits;     // bucket = key >> 19
constexpr int kHist2Bits = 10;                // second digit, counted among the bins of the threshold's bucket
constexpr int kHist2Bins = 1 << kHist2Bits;
constexpr int kHist2Shift = kKeyShift - kHist2Bits;

constexpr size_t kControlBytes = 4096;  // control block at the start of every workspace
constexpr int kCtlGaveUpWord = 1;       // u32 index of the fused kernels' give-up word inside the control block

// The fused transforms (fused.hip) take chunk lengths 2^16 .. 2^20 and address three turn buffers of 4 MiB per XCD
// inside the intermediate's region, so they take calls whose own intermediate is at least that large (96 MiB: about
// 25 million samples); smaller calls keep the per-pass kernels and their workspace stays what those need.
constexpr size_t kFusedScratchBytes = (size_t)8 * 3 * 64 * 8192 * 8;
static inline bool fused_shape(int logL, size_t C)
{
    const int logM = logL - 1;
    return logM >= 15 && logM <= 19 && (C << logL) * 4 >= kFusedScratchBytes;
}

// The receiver's kernels store one verdict per record, and the call's first kernel leaves this note in words 2..5 of the
// control block: how many there are, where (bytes from the workspace's start; calls with many short chunks have them
// beyond 16 GiB), and a magic word.  So no earlier kernel has to clear a status word before a record raises it.
// fftsp_device_status looks at both.
struct StatusNote {
    uint32_t count, low, high;  // low, high: the offset's halves
};
inline StatusNote status_note(size_t count, size_t offset)
{
    return StatusNote{(uint32_t)count, (uint32_t)offset, (uint32_t)((uint64_t)offset >> 32)};
}
constexpr uint32_t kStatusNoteMagic = 0x46535653u;
constexpr int kNoteWord = 2, kNoteWords = 4;  // of the control block
// word i of it, for these four
__host__ __device__ inline uint32_t note_word(const StatusNote& n, int i)
{
    switch (i - kNoteWord) {
        case 0: return n.count;
        case 1: return n.low;
        case 2: return n.count ? kStatusNoteMagic : 0u;
        default: return n.high;
    }
}

// Where everything lives inside the caller's workspace (byte offsets, 256-aligned).
struct Workspace {
    size_t status;    // u32[1024] control block: word 0 = device status, word 1 = "the fused transform gave up",
                      //           words 2..5 = where per-record verdicts are,
                      //           from word 32 on the hand-over counters of the fused kernels (fused.hip)
    size_t hist;      // u32[C][kHistBins]         (directly after status: one fill zeroes both)
    size_t sel;       // u32[C][8]  bstar, need, tau, quota, pbase, vmax, -, -
    size_t tinfo;     // u32[C][Tn][4]  n_def, vmax_def, n_cand, -
    size_t tscan;     // u32[C][Tn][2]  first rank of the tile, equal-key count before the tile
                      //                (receiver: u32[C] verdicts)
    size_t cand;      // uint2[C][Tn*kTile]  (key, max component bits) of threshold-bucket bins, tile-ordered
                      //                     (shares its bytes with mid)
    size_t prefix;    // u32[C][ceil(W/16)]  set bits before each group of 16 bitmap words (decode)
    size_t spec;      // float2[C][padded_bins(L)]  spectrum, each chunk on a 128-byte boundary
                      //                        (receivers that make none: the bitmaps' table, uint2[C][M/32 + 2])
    size_t mid;       // float2[C][L/2] intermediate of the two-pass FFT
    size_t total;
};

static inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
static inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Per-tensor mode, tensors longer than one workgroup takes: every launch covers up to kMaxLongTensors of them, each a
// single chunk of its own length 2^(logM+1).  What the kernels need to know about them travels by value as a kernel
// argument (no host-to-device copy to order against the stream).
constexpr int kMaxLongTensors = 64;
constexpr int kLongUnitLog = 15;  // the shortest has 2^15 complex values; their work areas are counted in these
struct LongTensor {
    uint64_t goff;    // element offset of its first sample in the gradient
    uint64_t roff;    // byte offset of its record from the first record of the stream
    uint32_t glen;    // samples present; the rest of the chunk is zero
    uint32_t kept;    // kept bins
    uint32_t stride;  // record bytes
    uint16_t base;    // units of 2^kLongUnitLog complex values of the launch's tensors before it
    uint8_t logM, pad;
};
// first workgroup of every tensor's share of a launch over tensors first .. first + count - 1
struct LongStarts {
    uint16_t at[kMaxLongTensors];
    uint32_t first, count;
};
struct LongTable {
    LongTensor t[kMaxLongTensors];
    LongStarts tiles;  // the codec kernels' share: a workgroup per tile of bins
};
// a launch set of the long tensors (host)
struct LongBatch {
    LongTable tab;
    uint32_t count, units;  // tensors, units of work area
};
// A few of them, as many as there is room for beside a table of shorter ones in a launch's arguments (with one more the receiver's are too many: FFTSP_LAUNCH).  at[i]: the first workgroup of tensor i's share.
// Sender and receiver in us, up to twelve / up to nineteen: random sets of 30 tensors 207.8 / 188.0, 40 182.6 / 169.1, 50 192.9 / 180.6 and 220.6 / 200.9.
// In launches of their own / there, twenty and twenty-two: of 40 k beside 60 of 9 k 83.2 / 74.4 and 83.9 / 77.9, of 2^17 beside 20 of 300 83.2 / 81.0 and 84.8 / 82.3, of 300 k 144 / 140 and 147 / 144.
constexpr int kFewLong = 22;
struct FewLong {
    LongTensor t[kFewLong];
    uint16_t at[kFewLong];
    uint32_t count;
};
// The first workgroups of tensors from .. end - 1 of a launch, wgs(logM) workgroups to each; returns how many in all.
template <typename Wgs>
uint32_t first_workgroups(const LongBatch& b, uint32_t from, uint32_t end, uint16_t* at, Wgs&& wgs)
{
    uint32_t sum = 0;
    for (uint32_t i = from; i < end; ++i) {
        at[i - from] = (uint16_t)sum;
        sum += wgs((int)b.tab.t[i].logM);
    }
    return sum;
}
template <typename Wgs>
uint32_t long_starts(const LongBatch& b, uint32_t from, uint32_t end, LongStarts* at, Wgs&& wgs)
{
    at->first = from;
    at->count = end - from;
    return first_workgroups(b, from, end, at->at, wgs);
}
// where tensor i of a launch finds its part of the work areas
__host__ __device__ inline size_t long_mid(const LongTensor& t) { return (size_t)t.base << kLongUnitLog; }
__host__ __device__ inline size_t long_spec(const LongTensor& t, uint32_t i) { return long_mid(t) + 16u * i; }
__host__ __device__ inline uint32_t long_tile(const LongTensor& t, uint32_t i) { return ((uint32_t)t.base << (kLongUnitLog - 11)) + i; }
__host__ __device__ inline uint32_t long_group(const LongTensor& t, uint32_t i) { return ((uint32_t)t.base << (kLongUnitLog - 9)) + i; }
__host__ __device__ inline int long_pair_log(const LongTensor& t) { return (t.logM + 1) / 2; }
static_assert(kTile == 1 << 11, "tiles of a tensor: M / 2^11 whole ones and one for the Nyquist bin");
// kernel parameter that is a LongTable in per-tensor launches and nothing otherwise
template <bool TABLE>
struct TableArg {
};
template <>
struct TableArg<true> {
    LongTable t;
};
template <bool TABLE>
inline TableArg<TABLE> table_arg(const LongBatch* b)
{
    TableArg<TABLE> a;
    if constexpr (TABLE) a.t = b->tab;
    return a;
}

// Several senders' packed streams decoded into one spectrum (receiver under an allgather).
constexpr int kMaxPeers = 32;
struct PeerList {
    const uint8_t* p[kMaxPeers];  // first record of each peer's stream
};
// Extra workspace behind the ordinary one: per peer the group prefixes of its bitmaps and its header verdicts.
struct PeerWorkspace {
    size_t prefix;  // u32[P][C][ceil(W/16)]
    size_t verd;    // u32[P][C]
    size_t total;   // end of the whole workspace
};

static inline uint32_t tiles_per_chunk(uint32_t L) { return ((L / 2 + 1) + kTile - 1) / kTile; }
// chunk stride of the codec's own spectrum buffer, in complex bins: L/2+1 rounded up to a 128-byte multiple
static inline uint32_t padded_bins(uint32_t L) { return (L / 2 + 1 + 15u) & ~15u; }

// What a chunk's record describes: L/2+1 frequency bins, or (time-domain Top-k) the L samples themselves.
static inline uint32_t codec_bins(uint32_t L, int time_domain) { return time_domain ? L : L / 2 + 1; }
static inline uint32_t codec_tiles(uint32_t L, int time_domain)
{
    return (codec_bins(L, time_domain) + kTile - 1) / kTile;
}

// time_domain != 0: no spectrum and no FFT intermediate (the codec kernels read and write the gradient itself)
static inline Workspace make_workspace(size_t C, uint32_t L, int time_domain = 0)
{
    Workspace w;
    size_t B = codec_bins(L, time_domain), Tn = codec_tiles(L, time_domain), W = (B + 31) / 32;
    size_t off = 0;
    w.status = off; off += kControlBytes;
    w.hist = off;   off = align256(off + C * kHistBins * 4);
    w.sel = off;    off = align256(off + C * 8 * 4);
    w.tinfo = off;  off = align256(off + C * Tn * 16);
    w.tscan = off;  off = align256(off + C * Tn * 8);
    // The candidate list and the two-pass intermediate are never alive together (the sender's transform has
    // finished before the first candidate is written; the receiver has no candidates): one region serves both.
    const size_t cand_bytes = C * Tn * kTile * 8, mid_bytes = time_domain ? 0 : C * (size_t)L * 4;
    w.cand = off;
    w.mid = off;    off = align256(off + (cand_bytes > mid_bytes ? cand_bytes : mid_bytes));
    w.prefix = off; off = align256(off + C * W * 4);
    w.spec = off;   off = align256(off + (time_domain ? 0 : C * (size_t)padded_bins(L) * 8));
    w.total = off;
    return w;
}

// the same for a launch set of long tensors
static inline Workspace make_long_workspace(const LongBatch& b)
{
    Workspace w;
    const size_t values = (size_t)b.units << kLongUnitLog, tiles = (values >> 11) + b.count;
    size_t off = 0;
    w.status = off; off += kControlBytes;
    w.hist = off;   off = align256(off + b.count * (size_t)kHistBins * 4);
    w.sel = off;    off = align256(off + b.count * 8 * 4);
    w.tinfo = off;  off = align256(off + tiles * 16);
    w.tscan = off;  off = align256(off + tiles * 8);
    w.cand = off;
    w.mid = off;    off = align256(off + tiles * kTile * 8);
    w.prefix = off; off = align256(off + ((values >> 5) + b.count) * 4);  // as above: more than the groups take
    w.spec = off;   off = align256(off + (values + 16 * (size_t)b.count) * 8);
    w.total = off;
    return w;
}

// Where bin j of a chunk sits inside the chunk's spectrum.  pair_log = 0: natural order (the layout of the
// stage-level entry points).  pair_log = log2(N1) > 0: the two-pass FFT's own "paired" order, in which each run
// of N1 bins stores bin k1 next to bin N1-k1 (position 2*k1 / 2*k1+1; position 1 holds k1 = N1/2), so that the
// rows the real-FFT split combines are one 128-byte run for the FFT passes.  Bin L/2 keeps index L/2.
__device__ __forceinline__ uint32_t spec_index(uint32_t j, int pair_log)
{
    if (pair_log == 0) return j;
    const uint32_t N1 = 1u << pair_log, k1 = j & (N1 - 1u), hi = j - k1;
    const uint32_t pos = k1 < N1 / 2 ? 2u * k1 : (k1 == N1 / 2 ? 1u : 2u * (N1 - k1) + 1u);
    return hi + pos;
}

// Optional per-kernel event timing (prof.hip).
namespace prof {
bool enabled();
int begin(const char* name, hipStream_t s);
void end(int id, hipStream_t s);
void enable(bool on);
std::string report();
}  // namespace prof

// bytes of a kernel's arguments
template <typename... A>
constexpr size_t argument_bytes(void (*)(A...))
{
    size_t at = 0;
    ((at = (at + alignof(A) - 1) / alignof(A) * alignof(A) + sizeof(A)), ...);
    return at;
}
// Launch `kernel` and, when profiling is on, bracket it with events under `name`.
#define FFTSP_LAUNCH(name, kernel, grid, block, lds, stream, ...)                    \
    do {                                                                             \
        static_assert(::fftsp::argument_bytes(std::decay_t<decltype(kernel)>{}) <= 4096, "kernel arguments are at most 4 KiB"); \
        const int fftsp_prof_id_ = ::fftsp::prof::enabled() ? ::fftsp::prof::begin(name, stream) : -1; \
        hipLaunchKernelGGL(kernel, grid, block, lds, stream, __VA_ARGS__);           \
        if (fftsp_prof_id_ >= 0) ::fftsp::prof::end(fftsp_prof_id_, stream);         \
    } while (0)

// per-device tables; returns hipSuccess or the failing HIP error
hipError_t get_tables(Tables* out);

// FFT launchers of the two-pass chunk lengths, 2^16 and up (fft.hip).  Chunk c covers in[c*L, min(n, (c+1)*L)), zero beyond n.
// spec: chunk c's L/2+1 bins start at spec + 2*c*sstride floats (sstride in complex bins: L/2+1 for the dense
// layout of the stage-level entry points, a multiple of 16 inside the codec so that every chunk starts on a
// 128-byte line); mid: C*L floats of scratch.
// hist (optional): u32[C][kHistBins]; the kernels clear zero_words words at zero_ptr (covering hist and the status
// words) and fill hist.  pair_spec != 0 (exactly when hist is given): the spectrum is written in paired order and
// *pair_log receives log2(N1), otherwise 0.
// only_if (optional, two-pass sizes): device word; the kernels return at once unless it is non-zero
hipError_t launch_rfft(const float* in, size_t n, int logL, size_t C, float* spec, uint32_t sstride, float2* mid,
                       Tables t, uint32_t* hist, uint32_t* zero_ptr, size_t zero_words, int pair_spec,
                       int* pair_log, hipStream_t s, const uint32_t* only_if = nullptr);
// log2(N1) of the two-pass factorisation for chunk length 2^logL (2^15 and up; 2^15 in the half-precision variant only)
int fft_pair_log(int logL);
// pair_spec != 0: the spectrum is in paired order; the output is gain/L times the plain sum
hipError_t launch_irfft(const float* spec, uint32_t sstride, size_t n, int logL, size_t C, float* out, float2* mid,
                        Tables t, int pair_spec, float gain, hipStream_t s, const uint32_t* only_if = nullptr);
// The same for a launch set of tensors of different lengths, paired order; spectra and intermediates lie as long_spec and
// long_mid say.
hipError_t launch_rfft_long(const float* in, const LongBatch& b, float2* spec, float2* mid, Tables t, uint32_t* hist,
                            uint32_t* zero_ptr, size_t zero_words, hipStream_t s);
// its second pass alone, where something else has filled mid and cleared what launch_rfft_long clears
hipError_t launch_rfft_b_long(const LongBatch& b, float2* spec, const float2* mid, Tables t, uint32_t* hist, hipStream_t s);
hipError_t launch_irfft_long(const float2* spec, const LongBatch& b, float* out, float2* mid, Tables t, hipStream_t s);
// Their second kernels alone (pass A), where something else has filled mid.  half: mid holds binary16 pairs.
hipError_t launch_inverse_a(const float2* mid, int logM, size_t C, float* out, size_t n, Tables t, float gain, int half, hipStream_t s,
                            const uint32_t* only_if = nullptr);
hipError_t launch_inverse_a_long(const float2* mid, const LongBatch& b, float* out, Tables t, hipStream_t s);
// A first-pass sum of N1 terms is about sqrt(N2) times smaller than a spectrum value, an unnormalised inverse second-pass sum
// about sqrt(N2) times larger: the half-precision variant's stored intermediate is lifted (lowered) by 2^(log2 N2 / 2) so that
// it sits where the caller's scale put the spectrum.  Powers of two: exact.
inline float half_lift(int logM) { return (float)(1u << (logM / 2 / 2)); }

// Fused two-pass transforms whose intermediate stays in the L2 caches (fused.hip).  They need the control block
// zeroed beforehand (launch_zero_control) and the per-pass kernels enqueued behind them with only_if = the give-up
// word, which redo the transform if the fused kernel could not finish.
struct FusedKnobs {
    int enabled;          // 0: never take the fused kernels
    uint32_t spin_limit;  // polls before a hand-over wait gives up
};
FusedKnobs fused_knobs();  // defaults overridden by the FFTSP_FUSED* environment variables (read at every call)
bool fused_applies(int logL, size_t C);
// spec: the codec's own buffer (paired order); hist: u32[C][kHistBins], already zero; ctl: the control block, zero
hipError_t launch_fused_rfft(const float* in, size_t n, int logL, size_t C, float2* spec, uint32_t sstride,
                             float2* scratch, Tables t, uint32_t* hist, uint32_t* ctl, const FusedKnobs& knobs,
                             hipStream_t s);
// the receiver's transform: spec is the codec's own decoded spectrum (paired order); ctl: the control block, zero
hipError_t launch_fused_irfft(const float2* spec, uint32_t sstride, size_t n, int logL, size_t C, float* out,
                              float2* scratch, Tables t, float gain, uint32_t* ctl, const FusedKnobs& knobs,
                              hipStream_t s);
// zeroes the control block and the histograms behind it (one fill)
hipError_t launch_zero_control(uint8_t* ws_base, const Workspace& w, size_t C, hipStream_t s);

// Half-precision variant: chunk lengths of the two-pass FFT only (2^15 and up); spec and mid are the codec's own
// buffers, read and written as binary16 pairs (sstride in complex values); the histogram is always produced.
hipError_t launch_rfft_half(const float* in, size_t n, int logL, size_t C, void* spec, uint32_t sstride, void* mid,
                            Tables t, uint32_t* hist, uint32_t* zero_ptr, size_t zero_words, float in_scale,
                            int* pair_log, hipStream_t s);
hipError_t launch_irfft_half(const void* spec, uint32_t sstride, size_t n, int logL, size_t C, float* out, void* mid,
                             Tables t, float gain, hipStream_t s);

// Codec launchers (codec.hip).
struct CodecArgs {
    size_t C;           // chunks
    uint32_t L;         // chunk length
    uint32_t k;         // kept bins per chunk
    int bits, m;        // code width, mantissa width
    size_t S;           // record stride in bytes
    uint32_t word3;     // 4th word of every record header
    uint32_t static_vmax;  // != 0: bit pattern of the caller's fixed range maximum (instead of the largest survivor)
    uint32_t sstride;   // distance between consecutive chunks' spectra, in complex bins
    const LongBatch* tab;  // per-tensor launches: the tensors (host pointer), C of them; else nullptr.  C, L, k, S, word3
                           // and sstride are then not used
    int time_domain;    // != 0: records describe the gradient's samples; `spec` of the launchers is the gradient
    size_t n;           // time domain: samples in the gradient (the last chunk may be short)
    int half;           // != 0: `spec` holds binary16 pairs (half-precision variant; two-pass chunk lengths only)
    int hdr_scale;      // stream header word 12: log2 of the factor on the spectrum (half-precision variant), else 0
    int pair_log;       // 0: spectrum in natural bin order; log2(N1): paired order (see spec_index)
    // stream header (written iff write_header)
    int write_header;
    uint64_t hdr_n;
    uint32_t hdr_L, hdr_C, hdr_k, hdr_S;
    float hdr_theta;
};
static inline PeerWorkspace make_peer_workspace(const Workspace& w, size_t C, uint32_t L, int npeers)
{
    PeerWorkspace pw;
    const size_t B = (size_t)L / 2 + 1, W = (B + 31) / 32, G = (W + 15) / 16;
    size_t off = w.total;
    pw.prefix = off; off = align256(off + (size_t)npeers * C * G * 4);
    pw.verd = off;   off = align256(off + (size_t)npeers * C * 4);
    pw.total = off;
    return pw;
}

// hist_ready != 0: the status words are cleared and the per-chunk histograms already hold the keys' top digit
hipError_t launch_encode(const float* spec, const CodecArgs& a, uint8_t* stream_base, uint8_t* records,
                         uint8_t* ws_base, const Workspace& w, int hist_ready, hipStream_t s);

// verdicts: u32[C].  note (optional): this launch clears the control block and leaves the note there (the first one of a
// call, or the only one).
hipError_t launch_decode(const uint8_t* stream_base, const uint8_t* records, const CodecArgs& a, float* spec,
                         uint8_t* ws_base, const Workspace& w, int check_header, uint32_t* verdicts, const StatusNote* note,
                         hipStream_t s);

// npeers streams (each: 64-byte header + records) summed bin by bin, in list order, into spec
hipError_t launch_decode_peers(const PeerList& streams, int npeers, const CodecArgs& a, float* spec, uint8_t* ws_base,
                               const Workspace& w, const PeerWorkspace& pw, hipStream_t s);

}  // namespace fftsp

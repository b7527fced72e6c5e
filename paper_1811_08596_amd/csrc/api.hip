// C ABI of libfftsp.so (see include/fftsp.h): argument checks, workspace carving, launch order.
#include "../../include/fftsp.h"
#include "chunk.h"
#include "internal.h"
#include "receive.h"
#include "short.h"
#include "twiddle_table.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

namespace fftsp {

namespace {
// Compile-time tables in device memory (twiddle_table.h): one copy per device, loaded with the code object.
// (not declared const: a const device variable that no device code names is dropped from the code object, and
// the host-side lookup of its address then finds nothing)
static __device__ twtab::Table g_tw_hi = twtab::make_table<11>();
static __device__ twtab::Table g_tw_lo = twtab::make_table<22>();
static_assert(sizeof(twtab::Pair) == sizeof(float2), "table entries are read as float2");

struct DeviceTables {
    bool ready = false;
    Tables t{nullptr, nullptr};
};
constexpr int kMaxDevices = 64;
DeviceTables g_tables[kMaxDevices];
std::mutex g_mutex;
}  // namespace

// Looks up this device's addresses of the two tables once; allocates nothing and enqueues nothing.
hipError_t get_tables(Tables* out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceTables& d = g_tables[dev];
    if (!d.ready) {
        void *hi = nullptr, *lo = nullptr;
        e = hipGetSymbolAddress(&hi, HIP_SYMBOL(g_tw_hi));
        if (e == hipSuccess) e = hipGetSymbolAddress(&lo, HIP_SYMBOL(g_tw_lo));
        if (e != hipSuccess) return e;
        d.t.hi = static_cast<const float2*>(hi);
        d.t.lo = static_cast<const float2*>(lo);
        d.ready = true;
    }
    *out = d.t;
    return hipSuccess;
}

namespace {

int log2_exact(uint32_t v)
{
    if (v == 0 || (v & (v - 1))) return -1;
    int l = 0;
    while ((1u << l) < v) ++l;
    return l;
}

int check_len(uint32_t L)
{
    const int l = log2_exact(L);
    if (l < kMinLogL || l > kMaxLogL) return -1;
    return l;
}

bool theta_ok(float t) { return t >= 0.0f && t <= 1.0f; }  // false for NaN

uint32_t kept(uint32_t L, float theta)
{
    const double B = (double)(L / 2 + 1);
    double k = std::floor((double)theta * B + 0.5);
    if (k < 0) k = 0;
    if (k > B) k = B;
    return (uint32_t)k;
}

int mantissa(int bits)
{
    if (bits == 32) return 23;
    if (bits < 3 || bits > 16) return -1;
    const int e = bits <= 6 ? 3 : (bits <= 12 ? 4 : 5);
    const int m = bits - 1 - e;
    return m < 1 ? 1 : m;
}

size_t record_stride(uint32_t L, uint32_t k, int bits)
{
    const size_t B = (size_t)L / 2 + 1, W = (B + 31) / 32;
    const size_t code_words = ((size_t)2 * k * (size_t)bits + 31) / 32;
    return (16 + 4 * W + 4 * code_words + 15) & ~(size_t)15;
}

constexpr size_t kStreamHeader = 64;


uint32_t segment_length(size_t size)
{
    uint32_t L = 32;
    while ((size_t)L < size && L < (1u << 31)) L <<= 1;
    return L;
}

struct Plan {
    size_t n, C;
    uint32_t L, k;
    int logL, bits, m;
    size_t S;
    Workspace ws;
};

// common argument checks for the uniform-chunk entry points; theta/bits optional
int make_plan(Plan* p, size_t n, uint32_t L, const float* theta, const int* bits)
{
    if (n == 0) return FFTSP_EINVAL;
    p->logL = check_len(L);
    if (p->logL < 0) return FFTSP_EUNSUPPORTED;
    p->n = n;
    p->L = L;
    p->C = (n + L - 1) / L;
    p->k = 0;
    p->bits = 32;
    p->m = 23;
    if (theta) {
        if (!theta_ok(*theta)) return FFTSP_EINVAL;
        p->k = kept(L, *theta);
    }
    if (bits) {
        p->m = mantissa(*bits);
        if (p->m < 0) return FFTSP_EINVAL;
        p->bits = *bits;
    }
    p->S = record_stride(L, p->k, p->bits);
    p->ws = make_workspace(p->C, L);
    return FFTSP_OK;
}

CodecArgs codec_args(const Plan& p, float theta)
{
    CodecArgs a{};
    a.C = p.C;
    a.L = p.L;
    a.k = p.k;
    a.bits = p.bits;
    a.m = p.m;
    a.S = p.S;
    a.word3 = 0;
    a.sstride = p.L / 2 + 1;  // dense layout, natural bin order; the codec's own buffer overrides both
    a.pair_log = 0;
    a.write_header = 1;
    a.hdr_n = p.n;
    a.hdr_L = p.L;
    a.hdr_C = (uint32_t)p.C;
    a.hdr_k = p.k;
    a.hdr_S = (uint32_t)p.S;
    a.hdr_theta = theta;
    return a;
}

int hip_status(hipError_t e) { return e == hipSuccess ? FFTSP_OK : FFTSP_EHIP; }

// ---- time-domain Top-k: chunks of L samples are ranked, coded and packed as they are ----
// a chunk's selection runs in one workgroup that keeps per-tile state in LDS for up to 1025 tiles of 2048
constexpr int kTopkMaxLogL = 21;

uint32_t topk_kept(uint32_t L, float theta)
{
    double k = std::floor((double)theta * (double)L + 0.5);
    if (k < 0) k = 0;
    if (k > (double)L) k = (double)L;
    return (uint32_t)k;
}

size_t topk_record_stride(uint32_t L, uint32_t k, int bits)
{
    const size_t W = ((size_t)L + 31) / 32;
    const size_t code_words = ((size_t)k * (size_t)bits + 31) / 32;
    return (16 + 4 * W + 4 * code_words + 15) & ~(size_t)15;
}

int make_topk_plan(Plan* p, size_t n, uint32_t L, const float* theta, int bits)
{
    if (n == 0) return FFTSP_EINVAL;
    p->logL = check_len(L);
    if (p->logL < 0 || p->logL > kTopkMaxLogL) return FFTSP_EUNSUPPORTED;
    p->n = n;
    p->L = L;
    p->C = (n + L - 1) / L;
    p->k = 0;
    if (theta) {
        if (!theta_ok(*theta)) return FFTSP_EINVAL;
        p->k = topk_kept(L, *theta);
    }
    p->m = mantissa(bits);
    if (p->m < 0) return FFTSP_EINVAL;
    p->bits = bits;
    p->S = topk_record_stride(L, p->k, bits);
    p->ws = make_workspace(p->C, L, 1);
    return FFTSP_OK;
}

CodecArgs topk_args(const Plan& p, float theta)
{
    CodecArgs a = codec_args(p, theta);
    a.sstride = p.L;  // chunk c of the "spectrum" is the gradient's own samples [c*L, (c+1)*L)
    a.time_domain = 1;
    a.n = p.n;
    return a;
}

// quantizer options (Sec. 3.2.1): a chosen m replaces the default of the width, a static range replaces the
// per-chunk fit; q == nullptr keeps both defaults
int apply_quantizer(Plan* p, const fftsp_quantizer* q, uint32_t* static_vmax)
{
    *static_vmax = 0;
    if (!q) return FFTSP_OK;
    if (q->mantissa_bits != 0 && p->bits != 32) {
        if (q->mantissa_bits < 1 || q->mantissa_bits > p->bits - 1) return FFTSP_EINVAL;
        p->m = q->mantissa_bits;
    }
    const float r = q->range_max;
    if (!(r >= 0.0f) || std::isinf(r)) return FFTSP_EINVAL;
    if (r > 0.0f) std::memcpy(static_vmax, &r, sizeof(uint32_t));
    return FFTSP_OK;
}

// All chunks of one stream to units; verdicts go where the sender would keep its tile prefixes.
hipError_t decode_stream(const Plan& p, const uint8_t* in, const CodecArgs& a, float* units, uint8_t* ws, hipStream_t s)
{
    if (p.C > 0xffffffffu) return hipErrorInvalidValue;
    const StatusNote note = status_note(p.C, p.ws.tscan);
    return launch_decode(in, in + kStreamHeader, a, units, ws, p.ws, 1, reinterpret_cast<uint32_t*>(ws + p.ws.tscan), &note, s);
}

// The whole receiver of one stream without a spectrum, where there are kernels for it (short.h, receive.h); false: there are none.
bool receive_without_spectrum(const Plan& p, const uint8_t* in, const CodecArgs& a, float* out, float gain, uint8_t* ws, size_t verd, Tables t,
                              hipStream_t s, hipError_t* e)
{
    const int logM = p.logL - 1;
    const FusedKnobs knobs = fused_knobs();
    if (p.C > 0xffffffffu || (knobs.enabled && fused_applies(p.logL, p.C))) return false;
    uint32_t *ctl = reinterpret_cast<uint32_t*>(ws + p.ws.status), *verdicts = reinterpret_cast<uint32_t*>(ws + verd);
    float2* mid = reinterpret_cast<float2*>(ws + p.ws.mid);
    const StatusNote note = status_note(p.C, verd);
    if (short_decode(logM, p.C))
        *e = launch_short_decode(in, a, logM, mid, t, verdicts, ctl, note, s);
    else if (receive_applies(logM, p.C, p.bits))
        *e = launch_receive(in, a, logM, ws + p.ws.spec, mid, t, verdicts, ctl, note, s);
    else
        return false;
    if (*e == hipSuccess) *e = launch_inverse_a(mid, logM, p.C, out, p.n, t, gain, a.half, s);
    return true;
}

// The receiver for chunks that fit one workgroup; its per-record verdicts go to the workspace at byte offset `verd`.
hipError_t decompress_chunks(const Plan& p, const PeerList& streams, int npeers, int plain, const CodecArgs& a, float* out,
                             float gain, uint8_t* ws, size_t verd, Tables t, hipStream_t s)
{
    const size_t count = p.C * (size_t)npeers;
    if (count > 0xffffffffu) return hipErrorInvalidValue;
    const StatusNote note = status_note(count, verd);
    return launch_chunk_decompress(streams, npeers, plain, p.logL, a, out, p.n, gain, reinterpret_cast<uint32_t*>(ws + p.ws.status),
                                   note, reinterpret_cast<uint32_t*>(ws + verd), t, s);
}

// The receiver's inverse transform of the codec's own spectrum buffer (uniform chunks).  The decode kernels that
// ran before it on this stream have cleared the control block.
hipError_t inverse_of_decoded(const Plan& p, const float* spec, uint32_t sstride, int pair_log, float* out, uint8_t* ws,
                              Tables t, float gain, hipStream_t s)
{
    float2* mid = reinterpret_cast<float2*>(ws + p.ws.mid);
    const FusedKnobs knobs = fused_knobs();
    if (knobs.enabled && pair_log != 0 && fused_applies(p.logL, p.C)) {
        uint32_t* ctl = reinterpret_cast<uint32_t*>(ws + p.ws.status);
        hipError_t e = launch_fused_irfft(reinterpret_cast<const float2*>(spec), sstride, p.n, p.logL, p.C, out, mid, t,
                                          gain, ctl, knobs, s);
        if (e != hipSuccess) return e;
        // stand-by: the per-pass kernels redo the transform if the fused kernel gave up
        return launch_irfft(spec, sstride, p.n, p.logL, p.C, out, mid, t, 1, gain, s, ctl + kCtlGaveUpWord);
    }
    return launch_irfft(spec, sstride, p.n, p.logL, p.C, out, mid, t, pair_log != 0, gain, s);
}

}  // namespace
}  // namespace fftsp

using namespace fftsp;

extern "C" {

int fftsp_kept_per_chunk(uint32_t chunk_len, float theta, uint32_t* k_out)
{
    if (!k_out || !theta_ok(theta)) return FFTSP_EINVAL;
    if (check_len(chunk_len) < 0) return FFTSP_EUNSUPPORTED;
    *k_out = kept(chunk_len, theta);
    return FFTSP_OK;
}

int fftsp_mantissa_bits(int bits) { return mantissa(bits); }

size_t fftsp_packed_bytes(size_t n, uint32_t chunk_len, float theta, int bits)
{
    Plan p;
    if (make_plan(&p, n, chunk_len, &theta, &bits) != FFTSP_OK) return 0;
    return kStreamHeader + p.C * p.S;
}

size_t fftsp_workspace_bytes(size_t n, uint32_t chunk_len, int bits)
{
    Plan p;
    if (make_plan(&p, n, chunk_len, nullptr, &bits) != FFTSP_OK) return 0;
    return p.ws.total;
}

int fftsp_rfft(const float* d_grad, size_t n, uint32_t chunk_len, float* d_spec, void* d_workspace,
               size_t workspace_bytes, fftsp_stream_t stream)
{
    Plan p;
    int rc = make_plan(&p, n, chunk_len, nullptr, nullptr);
    if (rc) return rc;
    if (!d_grad || !d_spec || !d_workspace || !aligned16(d_grad) || !aligned16(d_spec) || !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (workspace_bytes < p.ws.total) return FFTSP_EWORKSPACE;
    Tables t;
    if (get_tables(&t) != hipSuccess) return FFTSP_EHIP;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (p.logL <= kChunkMaxLogL) return hip_status(launch_chunk_rfft(d_grad, n, p.logL, p.C, d_spec, p.L / 2 + 1, t, s));
    return hip_status(launch_rfft(d_grad, n, p.logL, p.C, d_spec, p.L / 2 + 1, reinterpret_cast<float2*>(ws + p.ws.mid), t,
                                  nullptr, nullptr, 0, 0, nullptr, s));
}

int fftsp_irfft(const float* d_spec, size_t n, uint32_t chunk_len, float* d_grad_out, void* d_workspace,
                size_t workspace_bytes, fftsp_stream_t stream)
{
    Plan p;
    int rc = make_plan(&p, n, chunk_len, nullptr, nullptr);
    if (rc) return rc;
    if (!d_grad_out || !d_spec || !d_workspace || !aligned16(d_grad_out) || !aligned16(d_spec) ||
        !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (workspace_bytes < p.ws.total) return FFTSP_EWORKSPACE;
    Tables t;
    if (get_tables(&t) != hipSuccess) return FFTSP_EHIP;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (p.logL <= kChunkMaxLogL) return hip_status(launch_chunk_irfft(d_spec, p.L / 2 + 1, n, p.logL, p.C, d_grad_out, t, s));
    return hip_status(launch_irfft(d_spec, p.L / 2 + 1, n, p.logL, p.C, d_grad_out, reinterpret_cast<float2*>(ws + p.ws.mid), t,
                                   0, 1.0f, s));
}

int fftsp_encode_spectrum_q(const float* d_spec, size_t n, uint32_t chunk_len, float theta, int bits, void* d_packed,
                          size_t packed_capacity, void* d_workspace, size_t workspace_bytes, const fftsp_quantizer* quantizer, fftsp_stream_t stream)
{
    Plan p;
    int rc = make_plan(&p, n, chunk_len, &theta, &bits);
    if (rc) return rc;
    uint32_t static_vmax = 0;
    rc = apply_quantizer(&p, quantizer, &static_vmax);
    if (rc) return rc;
    if (!d_spec || !d_packed || !d_workspace || !aligned16(d_spec) || !aligned16(d_packed) || !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (packed_capacity < kStreamHeader + p.C * p.S) return FFTSP_ENOSPC;
    if (workspace_bytes < p.ws.total) return FFTSP_EWORKSPACE;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    uint8_t* out = static_cast<uint8_t*>(d_packed);
    CodecArgs a = codec_args(p, theta);
    a.static_vmax = static_vmax;
    return hip_status(launch_encode(d_spec, a, out, out + kStreamHeader, ws, p.ws, 0,
                                    reinterpret_cast<hipStream_t>(stream)));
}

int fftsp_encode_spectrum(const float* d_spec, size_t n, uint32_t chunk_len, float theta, int bits, void* d_packed,
                          size_t packed_capacity, void* d_workspace, size_t workspace_bytes, fftsp_stream_t stream)
{
    return fftsp_encode_spectrum_q(d_spec, n, chunk_len, theta, bits, d_packed, packed_capacity, d_workspace, workspace_bytes, nullptr, stream);
}

int fftsp_decode_spectrum_q(const void* d_packed, size_t packed_bytes, size_t n, uint32_t chunk_len, float theta,
                          int bits, float* d_spec, void* d_workspace, size_t workspace_bytes, const fftsp_quantizer* quantizer, fftsp_stream_t stream)
{
    Plan p;
    int rc = make_plan(&p, n, chunk_len, &theta, &bits);
    if (rc) return rc;
    uint32_t static_vmax = 0;
    rc = apply_quantizer(&p, quantizer, &static_vmax);
    if (rc) return rc;
    (void)static_vmax;  // the receiver reads the range from the records; only m matters here
    if (!d_spec || !d_packed || !d_workspace || !aligned16(d_spec) || !aligned16(d_packed) || !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (packed_bytes < kStreamHeader + p.C * p.S) return FFTSP_EFORMAT;
    if (workspace_bytes < p.ws.total) return FFTSP_EWORKSPACE;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    const uint8_t* in = static_cast<const uint8_t*>(d_packed);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipError_t e = decode_stream(p, in, codec_args(p, theta), d_spec, ws, s);
    return hip_status(e);
}

int fftsp_decode_spectrum(const void* d_packed, size_t packed_bytes, size_t n, uint32_t chunk_len, float theta,
                          int bits, float* d_spec, void* d_workspace, size_t workspace_bytes, fftsp_stream_t stream)
{
    return fftsp_decode_spectrum_q(d_packed, packed_bytes, n, chunk_len, theta, bits, d_spec, d_workspace, workspace_bytes, nullptr, stream);
}

}  // extern "C"

// the sender proper, shared by the entry points that differ only in where the workspace comes from
static int compress_impl(const float* d_grad, size_t n, uint32_t chunk_len, float theta, int bits, void* d_packed,
                         size_t packed_capacity, void* d_workspace, size_t workspace_bytes,
                         const fftsp_quantizer* quantizer, hipStream_t s)
{
    Plan p;
    int rc = make_plan(&p, n, chunk_len, &theta, &bits);
    if (rc) return rc;
    uint32_t static_vmax = 0;
    rc = apply_quantizer(&p, quantizer, &static_vmax);
    if (rc) return rc;
    if (!d_grad || !d_packed || !d_workspace || !aligned16(d_grad) || !aligned16(d_packed) || !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (packed_capacity < kStreamHeader + p.C * p.S) return FFTSP_ENOSPC;
    if (workspace_bytes < p.ws.total) return FFTSP_EWORKSPACE;
    Tables t;
    if (get_tables(&t) != hipSuccess) return FFTSP_EHIP;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    uint8_t* out = static_cast<uint8_t*>(d_packed);
    float* spec = reinterpret_cast<float*>(ws + p.ws.spec);
    CodecArgs a = codec_args(p, theta);
    a.static_vmax = static_vmax;
    a.sstride = padded_bins(p.L);
    uint32_t* ctl = reinterpret_cast<uint32_t*>(ws + p.ws.status);
    if (p.logL <= kChunkMaxLogL)
        return hip_status(launch_chunk_compress(d_grad, n, p.logL, a, out, out + kStreamHeader, ctl, t, s));
    uint32_t* hist = reinterpret_cast<uint32_t*>(ws + p.ws.hist);
    float2* mid = reinterpret_cast<float2*>(ws + p.ws.mid);
    const FusedKnobs knobs = fused_knobs();
    hipError_t e;
    if (knobs.enabled && fused_applies(p.logL, p.C)) {
        // both passes in one kernel, the intermediate in the L2 caches (fused.hip); the per-pass kernels stand by
        // behind it and run only if it gave up (they then clear the histograms again, not the control block)
        e = launch_zero_control(ws, p.ws, p.C, s);
        if (e == hipSuccess)
            e = launch_fused_rfft(d_grad, n, p.logL, p.C, reinterpret_cast<float2*>(spec), a.sstride, mid, t, hist, ctl,
                                  knobs, s);
        if (e == hipSuccess)
            e = launch_rfft(d_grad, n, p.logL, p.C, spec, a.sstride, mid, t, hist, hist, p.C * kHistBins, 1,
                            &a.pair_log, s, ctl + kCtlGaveUpWord);
    } else {
        e = launch_rfft(d_grad, n, p.logL, p.C, spec, a.sstride, mid, t, hist, ctl,
                        (p.ws.hist - p.ws.status) / 4 + p.C * kHistBins, 1, &a.pair_log, s);
    }
    if (e == hipSuccess)
        e = launch_encode(spec, a, out, out + kStreamHeader, ws, p.ws, 1, s);
    return hip_status(e);
}

// Workspace of fftsp_compress_static: one array per device inside the code object.  Host code never uses the
// array's name as an address: the device address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[FFTSP_STATIC_SCRATCH_BYTES];
static void* g_scratch_ptr[64];
static std::mutex g_scratch_mutex;

static hipError_t static_scratch(void** out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

extern "C" {

int fftsp_compress_q(const float* d_grad, size_t n, uint32_t chunk_len, float theta, int bits, void* d_packed,
                   size_t packed_capacity, void* d_workspace, size_t workspace_bytes, const fftsp_quantizer* quantizer, fftsp_stream_t stream)
{
    return compress_impl(d_grad, n, chunk_len, theta, bits, d_packed, packed_capacity, d_workspace, workspace_bytes,
                         quantizer, reinterpret_cast<hipStream_t>(stream));
}

int fftsp_compress_static(const float* d_grad, size_t n, uint32_t chunk_len, float theta, int bits, void* d_packed,
                          size_t packed_capacity, fftsp_stream_t stream)
{
    // sizes first: a call that cannot fit is refused before the device is touched
    Plan p;
    const int rc = make_plan(&p, n, chunk_len, &theta, &bits);
    if (rc) return rc;
    if (p.ws.total > (size_t)FFTSP_STATIC_SCRATCH_BYTES) return FFTSP_EWORKSPACE;
    void* ws = nullptr;
    if (static_scratch(&ws) != hipSuccess) return FFTSP_EHIP;
    return compress_impl(d_grad, n, chunk_len, theta, bits, d_packed, packed_capacity, ws,
                         (size_t)FFTSP_STATIC_SCRATCH_BYTES, nullptr, reinterpret_cast<hipStream_t>(stream));
}

int fftsp_compress(const float* d_grad, size_t n, uint32_t chunk_len, float theta, int bits, void* d_packed,
                   size_t packed_capacity, void* d_workspace, size_t workspace_bytes, fftsp_stream_t stream)
{
    return fftsp_compress_q(d_grad, n, chunk_len, theta, bits, d_packed, packed_capacity, d_workspace, workspace_bytes, nullptr, stream);
}

int fftsp_decompress_q(const void* d_packed, size_t packed_bytes, float* d_grad_out, size_t n, uint32_t chunk_len,
                     float theta, int bits, void* d_workspace, size_t workspace_bytes, const fftsp_quantizer* quantizer, fftsp_stream_t stream)
{
    Plan p;
    int rc = make_plan(&p, n, chunk_len, &theta, &bits);
    if (rc) return rc;
    uint32_t static_vmax = 0;
    rc = apply_quantizer(&p, quantizer, &static_vmax);
    if (rc) return rc;
    (void)static_vmax;  // the receiver reads the range from the records; only m matters here
    if (!d_grad_out || !d_packed || !d_workspace || !aligned16(d_grad_out) || !aligned16(d_packed) ||
        !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (packed_bytes < kStreamHeader + p.C * p.S) return FFTSP_EFORMAT;
    if (workspace_bytes < p.ws.total) return FFTSP_EWORKSPACE;
    Tables t;
    if (get_tables(&t) != hipSuccess) return FFTSP_EHIP;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    const uint8_t* in = static_cast<const uint8_t*>(d_packed);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    float* spec = reinterpret_cast<float*>(ws + p.ws.spec);
    CodecArgs a = codec_args(p, theta);
    if (p.logL <= kChunkMaxLogL) {
        PeerList one{};
        one.p[0] = in;
        return hip_status(decompress_chunks(p, one, 1, 1, a, d_grad_out, 1.0f, ws, p.ws.sel, t, s));
    }
    a.sstride = padded_bins(p.L);
    a.pair_log = fft_pair_log(p.logL);
    hipError_t e;
    if (receive_without_spectrum(p, in, a, d_grad_out, 1.0f, ws, p.ws.tscan, t, s, &e)) return hip_status(e);
    e = decode_stream(p, in, a, spec, ws, s);
    if (e == hipSuccess) e = inverse_of_decoded(p, spec, a.sstride, a.pair_log, d_grad_out, ws, t, 1.0f, s);
    return hip_status(e);
}

int fftsp_decompress(const void* d_packed, size_t packed_bytes, float* d_grad_out, size_t n, uint32_t chunk_len,
                     float theta, int bits, void* d_workspace, size_t workspace_bytes, fftsp_stream_t stream)
{
    return fftsp_decompress_q(d_packed, packed_bytes, d_grad_out, n, chunk_len, theta, bits, d_workspace, workspace_bytes, nullptr, stream);
}

/* ---------------- receiver under an allgather: several peers' streams, one inverse transform ---------------- */

static int peer_list(PeerList* out, const void* const* d_packed, int npeers)
{
    if (!d_packed || npeers < 1) return FFTSP_EINVAL;
    if (npeers > kMaxPeers) return FFTSP_EUNSUPPORTED;
    for (int i = 0; i < kMaxPeers; ++i) out->p[i] = nullptr;
    for (int i = 0; i < npeers; ++i) {
        if (!d_packed[i] || !aligned16(d_packed[i])) return FFTSP_EINVAL;
        out->p[i] = static_cast<const uint8_t*>(d_packed[i]);
    }
    return FFTSP_OK;
}

size_t fftsp_workspace_bytes_accumulate(size_t n, uint32_t chunk_len, int bits, int npeers)
{
    Plan p;
    if (npeers < 1 || npeers > kMaxPeers || make_plan(&p, n, chunk_len, nullptr, &bits) != FFTSP_OK) return 0;
    return make_peer_workspace(p.ws, p.C, p.L, npeers).total;
}

int fftsp_decode_accumulate_spectrum(const void* const* d_packed, int npeers, size_t packed_bytes, size_t n,
                                     uint32_t chunk_len, float theta, int bits, float* d_spec, void* d_workspace,
                                     size_t workspace_bytes, fftsp_stream_t stream)
{
    Plan p;
    int rc = make_plan(&p, n, chunk_len, &theta, &bits);
    if (rc) return rc;
    PeerList peers;
    rc = peer_list(&peers, d_packed, npeers);
    if (rc) return rc;
    if (!d_spec || !d_workspace || !aligned16(d_spec) || !aligned16(d_workspace)) return FFTSP_EINVAL;
    if (packed_bytes < kStreamHeader + p.C * p.S) return FFTSP_EFORMAT;
    const PeerWorkspace pw = make_peer_workspace(p.ws, p.C, p.L, npeers);
    if (workspace_bytes < pw.total) return FFTSP_EWORKSPACE;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    return hip_status(launch_decode_peers(peers, npeers, codec_args(p, theta), d_spec, ws, p.ws, pw,
                                          reinterpret_cast<hipStream_t>(stream)));
}

int fftsp_decompress_accumulate(const void* const* d_packed, int npeers, size_t packed_bytes, float scale,
                                float* d_grad_out, size_t n, uint32_t chunk_len, float theta, int bits,
                                void* d_workspace, size_t workspace_bytes, fftsp_stream_t stream)
{
    Plan p;
    int rc = make_plan(&p, n, chunk_len, &theta, &bits);
    if (rc) return rc;
    PeerList peers;
    rc = peer_list(&peers, d_packed, npeers);
    if (rc) return rc;
    if (!d_grad_out || !d_workspace || !aligned16(d_grad_out) || !aligned16(d_workspace) || !(scale == scale))
        return FFTSP_EINVAL;
    if (packed_bytes < kStreamHeader + p.C * p.S) return FFTSP_EFORMAT;
    const PeerWorkspace pw = make_peer_workspace(p.ws, p.C, p.L, npeers);
    if (workspace_bytes < pw.total) return FFTSP_EWORKSPACE;
    Tables t;
    if (get_tables(&t) != hipSuccess) return FFTSP_EHIP;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    float* spec = reinterpret_cast<float*>(ws + p.ws.spec);
    CodecArgs a = codec_args(p, theta);
    if (p.logL <= kChunkMaxLogL)
        return hip_status(decompress_chunks(p, peers, npeers, 0, a, d_grad_out, scale, ws, pw.verd, t, s));
    a.sstride = padded_bins(p.L);
    a.pair_log = fft_pair_log(p.logL);
    hipError_t e;
    // a sum of one: adding to zero changes nothing, there are no negative zeros among decoded values but the raw ones
    if (npeers == 1 && p.bits != 32 && receive_without_spectrum(p, peers.p[0], a, d_grad_out, scale, ws, pw.verd, t, s, &e))
        return hip_status(e);
    e = launch_decode_peers(peers, npeers, a, spec, ws, p.ws, pw, s);
    if (e == hipSuccess) e = inverse_of_decoded(p, spec, a.sstride, a.pair_log, d_grad_out, ws, t, scale, s);
    return hip_status(e);
}

/* ---------------- half-precision variant: binary16 between the passes and in the spectrum ---------------- */

namespace {
constexpr int kHalfMinLogL = 15;  // the two-pass FFT starts here; shorter chunks do not need the variant
bool half_scale_ok(int s) { return s >= -24 && s <= 24; }
}  // namespace

int fftsp_compress_h(const float* d_grad, size_t n, uint32_t chunk_len, float theta, int bits, int scale_log2,
                     void* d_packed, size_t packed_capacity, void* d_workspace, size_t workspace_bytes,
                     fftsp_stream_t stream)
{
    Plan p;
    int rc = make_plan(&p, n, chunk_len, &theta, &bits);
    if (rc) return rc;
    if (p.logL < kHalfMinLogL) return FFTSP_EUNSUPPORTED;
    if (!half_scale_ok(scale_log2)) return FFTSP_EINVAL;
    if (!d_grad || !d_packed || !d_workspace || !aligned16(d_grad) || !aligned16(d_packed) || !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (packed_capacity < kStreamHeader + p.C * p.S) return FFTSP_ENOSPC;
    if (workspace_bytes < p.ws.total) return FFTSP_EWORKSPACE;
    Tables t;
    if (get_tables(&t) != hipSuccess) return FFTSP_EHIP;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    uint8_t* out = static_cast<uint8_t*>(d_packed);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    CodecArgs a = codec_args(p, theta);
    a.sstride = padded_bins(p.L);
    a.half = 1;
    a.hdr_scale = scale_log2;
    hipError_t e = launch_rfft_half(d_grad, n, p.logL, p.C, ws + p.ws.spec, a.sstride, ws + p.ws.mid, t,
                                    reinterpret_cast<uint32_t*>(ws + p.ws.hist),
                                    reinterpret_cast<uint32_t*>(ws + p.ws.status),
                                    (p.ws.hist - p.ws.status) / 4 + p.C * kHistBins, std::ldexp(1.0f, scale_log2),
                                    &a.pair_log, s);
    if (e == hipSuccess)
        e = launch_encode(reinterpret_cast<const float*>(ws + p.ws.spec), a, out, out + kStreamHeader, ws, p.ws, 1, s);
    return hip_status(e);
}

int fftsp_decompress_h(const void* d_packed, size_t packed_bytes, float* d_grad_out, size_t n, uint32_t chunk_len,
                       float theta, int bits, int scale_log2, void* d_workspace, size_t workspace_bytes,
                       fftsp_stream_t stream)
{
    Plan p;
    int rc = make_plan(&p, n, chunk_len, &theta, &bits);
    if (rc) return rc;
    if (p.logL < kHalfMinLogL) return FFTSP_EUNSUPPORTED;
    if (!half_scale_ok(scale_log2)) return FFTSP_EINVAL;
    if (!d_grad_out || !d_packed || !d_workspace || !aligned16(d_grad_out) || !aligned16(d_packed) ||
        !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (packed_bytes < kStreamHeader + p.C * p.S) return FFTSP_EFORMAT;
    if (workspace_bytes < p.ws.total) return FFTSP_EWORKSPACE;
    Tables t;
    if (get_tables(&t) != hipSuccess) return FFTSP_EHIP;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    const uint8_t* in = static_cast<const uint8_t*>(d_packed);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    CodecArgs a = codec_args(p, theta);
    a.sstride = padded_bins(p.L);
    a.pair_log = fft_pair_log(p.logL);
    a.half = 1;
    a.hdr_scale = scale_log2;
    const float gain = std::ldexp(1.0f, -scale_log2);
    hipError_t e;
    if (receive_without_spectrum(p, in, a, d_grad_out, gain, ws, p.ws.tscan, t, s, &e)) return hip_status(e);
    e = decode_stream(p, in, a, reinterpret_cast<float*>(ws + p.ws.spec), ws, s);
    if (e == hipSuccess) e = launch_irfft_half(ws + p.ws.spec, a.sstride, n, p.logL, p.C, d_grad_out, ws + p.ws.mid, t, gain, s);
    return hip_status(e);
}

/* ---------------- time-domain Top-k: the same select / quantize / pack kernels, no transform ---------------- */

int fftsp_topk_kept_per_chunk(uint32_t chunk_len, float theta, uint32_t* k_out)
{
    if (!k_out || !theta_ok(theta)) return FFTSP_EINVAL;
    const int l = check_len(chunk_len);
    if (l < 0 || l > kTopkMaxLogL) return FFTSP_EUNSUPPORTED;
    *k_out = topk_kept(chunk_len, theta);
    return FFTSP_OK;
}

size_t fftsp_topk_packed_bytes(size_t n, uint32_t chunk_len, float theta, int bits)
{
    Plan p;
    if (make_topk_plan(&p, n, chunk_len, &theta, bits) != FFTSP_OK) return 0;
    return kStreamHeader + p.C * p.S;
}

size_t fftsp_topk_workspace_bytes(size_t n, uint32_t chunk_len, int bits)
{
    Plan p;
    if (make_topk_plan(&p, n, chunk_len, nullptr, bits) != FFTSP_OK) return 0;
    return p.ws.total;
}

int fftsp_topk_compress(const float* d_grad, size_t n, uint32_t chunk_len, float theta, int bits, void* d_packed,
                        size_t packed_capacity, void* d_workspace, size_t workspace_bytes, fftsp_stream_t stream)
{
    Plan p;
    int rc = make_topk_plan(&p, n, chunk_len, &theta, bits);
    if (rc) return rc;
    if (!d_grad || !d_packed || !d_workspace || !aligned16(d_grad) || !aligned16(d_packed) || !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (packed_capacity < kStreamHeader + p.C * p.S) return FFTSP_ENOSPC;
    if (workspace_bytes < p.ws.total) return FFTSP_EWORKSPACE;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    uint8_t* out = static_cast<uint8_t*>(d_packed);
    const CodecArgs a = topk_args(p, theta);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (p.logL <= kChunkMaxLogL)
        return hip_status(launch_topk_compress(d_grad, p.n, p.logL, a, out, out + kStreamHeader,
                                               reinterpret_cast<uint32_t*>(ws + p.ws.status), s));
    return hip_status(launch_encode(d_grad, a, out, out + kStreamHeader, ws, p.ws, 0, s));
}

int fftsp_topk_decompress(const void* d_packed, size_t packed_bytes, float* d_grad_out, size_t n, uint32_t chunk_len,
                          float theta, int bits, void* d_workspace, size_t workspace_bytes, fftsp_stream_t stream)
{
    Plan p;
    int rc = make_topk_plan(&p, n, chunk_len, &theta, bits);
    if (rc) return rc;
    if (!d_grad_out || !d_packed || !d_workspace || !aligned16(d_grad_out) || !aligned16(d_packed) ||
        !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (packed_bytes < kStreamHeader + p.C * p.S) return FFTSP_EFORMAT;
    if (workspace_bytes < p.ws.total) return FFTSP_EWORKSPACE;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    const uint8_t* in = static_cast<const uint8_t*>(d_packed);
    const CodecArgs a = topk_args(p, theta);
    return hip_status(decode_stream(p, in, a, d_grad_out, ws, reinterpret_cast<hipStream_t>(stream)));
}

/* ---------------- per-tensor variant: one single-chunk codec per segment ---------------- */

static int segments_ok(const size_t* off, int nseg)
{
    if (!off || nseg <= 0) return FFTSP_EINVAL;
    for (int i = 0; i < nseg; ++i) {
        if (off[i + 1] <= off[i]) return FFTSP_EINVAL;
        if (off[i + 1] - off[i] > ((size_t)1 << kMaxLogL)) return FFTSP_EUNSUPPORTED;
    }
    return FFTSP_OK;
}

size_t fftsp_packed_bytes_segments(const size_t* seg_offsets, int nseg, float theta, int bits)
{
    if (segments_ok(seg_offsets, nseg) != FFTSP_OK || !theta_ok(theta) || mantissa(bits) < 0) return 0;
    size_t total = kStreamHeader;
    for (int i = 0; i < nseg; ++i) {
        const uint32_t L = segment_length(seg_offsets[i + 1] - seg_offsets[i]);
        total += record_stride(L, kept(L, theta), bits);
    }
    return total;
}

// The longer tensors run in launch sets of at most kMaxLongTensors (the per-launch table), together at most 2^26 padded
// samples, so that the workspace stays a small multiple of the largest tensor.
constexpr uint32_t kMaxLongUnits = (1u << 26) >> (kLongUnitLog + 1);

// A launch of tensors that fit one workgroup each (chunk.h).
struct TensorLaunch {
    uint32_t pieces;
    int top_logL;
    TensorTable tab;
};

// How a per-tensor call is launched: the tensors of up to 2^kChunkMaxLogL samples in as few launches as the table
// allows, longest first; the longer ones in launch sets of any lengths, shortest first.
// Records keep tensor order in the stream: tensor i's record starts rec_off[i] bytes after the stream header.
struct SegmentPlan {
    std::vector<TensorLaunch> shorts;
    std::vector<LongBatch> longs;
    size_t short_count = 0;
};
static SegmentPlan plan_segments(const size_t* off, int nseg, float theta, int bits, bool with_tables)
{
    std::vector<uint32_t> len(nseg);
    std::vector<size_t> rec_off(nseg);
    std::vector<int> order(nseg);
    size_t ro = 0;
    for (int i = 0; i < nseg; ++i) {
        len[i] = segment_length(off[i + 1] - off[i]);
        rec_off[i] = ro;
        if (with_tables) ro += record_stride(len[i], kept(len[i], theta), bits);
        order[i] = i;
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return len[a] < len[b]; });
    SegmentPlan out;
    size_t first_long = 0;
    while (first_long < order.size() && len[order[first_long]] <= (1u << kChunkMaxLogL)) ++first_long;
    out.short_count = first_long;
    if (with_tables) {
        uint32_t used = 0;  // entries of the open launch
        for (size_t j = first_long; j-- > 0;) {  // longest first
            const int i = order[j];
            const int logL = log2_exact(len[i]);
            if (out.shorts.empty() || used == (uint32_t)kMaxTensors) {
                out.shorts.emplace_back();
                TensorLaunch& l = out.shorts.back();
                l.pieces = 0;
                l.top_logL = logL;
                l.tab.base = (uint32_t)(first_long - 1 - j);
                for (int g = 0; g < kChunkMaxLogL - 4; ++g) {
                    const uint32_t L = 1u << (g + 5);
                    l.tab.kept[g] = kept(L, theta);
                    l.tab.stride[g] = (uint32_t)record_stride(L, l.tab.kept[g], bits);
                }
                used = 0;
            }
            TensorLaunch& l = out.shorts.back();
            l.tab.goff[used] = off[i];
            l.tab.glen[used] = (uint32_t)(off[i + 1] - off[i]);
            l.tab.roff[used] = rec_off[i];
            TensorPiece* last = l.pieces ? &l.tab.piece[l.pieces - 1] : nullptr;
            if (last && last->logm == logL - 1 && last->count < tensors_per_workgroup(logL))
                ++last->count;
            else
                l.tab.piece[l.pieces++] = TensorPiece{(uint8_t)used, 1, (uint8_t)(logL - 1), 0};
            ++used;
        }
    }
    for (size_t j = first_long; j < order.size(); ++j) {
        const int i = order[j], logM = log2_exact(len[i]) - 1;
        const uint32_t units = 1u << (logM - kLongUnitLog);
        if (out.longs.empty() || out.longs.back().count == (uint32_t)kMaxLongTensors || out.longs.back().units + units > kMaxLongUnits) {
            out.longs.emplace_back();
            out.longs.back().count = out.longs.back().units = 0;
        }
        LongBatch& b = out.longs.back();
        LongTensor& x = b.tab.t[b.count];
        x.goff = off[i];
        x.roff = rec_off[i];
        x.glen = (uint32_t)(off[i + 1] - off[i]);
        x.kept = with_tables ? kept(len[i], theta) : 0u;
        x.stride = with_tables ? (uint32_t)record_stride(len[i], x.kept, bits) : 0u;
        x.base = (uint16_t)b.units;
        x.logM = (uint8_t)logM;
        x.pad = 0;
        b.tab.tiles.at[b.count] = (uint16_t)long_tile(x, b.count);
        b.tab.tiles.first = 0;
        b.units += units;
        b.tab.tiles.count = ++b.count;
    }
    return out;
}

// The tensors that fit a workgroup each and the longer ones are independent, so the former run on a stream of the library's
// own that forks from and joins back into the caller's through events.  The call stays one unit of work on the caller's
// stream and can be captured into a graph.
struct SideStream {
    bool ready = false;
    hipStream_t s;
    hipEvent_t fork, join;
};
static SideStream g_side[64];
static std::mutex g_side_mutex;  // held while a call enqueues: the events are shared by all calls on a device

// where the tensors' verdicts are: behind the longer ones' workspace, or behind a control block of their own
static size_t segment_verdicts(const SegmentPlan& plan)
{
    size_t most = kControlBytes;
    for (const LongBatch& b : plan.longs) most = std::max(most, make_long_workspace(b).total);
    return align256(most);
}

size_t fftsp_workspace_bytes_segments(const size_t* seg_offsets, int nseg, int bits)
{
    if (segments_ok(seg_offsets, nseg) != FFTSP_OK || mantissa(bits) < 0) return 0;
    const SegmentPlan plan = plan_segments(seg_offsets, nseg, 0.5f, bits, false);
    return segment_verdicts(plan) + align256((size_t)nseg * 4);
}

}  // extern "C" (a template cannot have C linkage)

// The capture `s` is being recorded into: its id, 0 if none, ~0 if the capture is broken.
static hipError_t capture_of(hipStream_t s, unsigned long long* id)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    unsigned long long i = 0;
    const hipError_t e = hipStreamGetCaptureInfo(s, &st, &i);
    if (e != hipSuccess) return e;
    *id = st == hipStreamCaptureStatusNone ? 0ull : (st == hipStreamCaptureStatusActive ? i : ~0ull);
    return hipSuccess;
}

// side(stream) and main(stream) enqueue independent work; main's stream is the caller's.
// The side stream belongs to the device, not to a caller.  A caller that records its stream into a graph pulls it into that
// capture until it ends, so a call falls back to the caller's stream alone (the same result, one after the other) when the
// side stream is being recorded into a capture other than the caller's own, and when it does not exist yet and the caller is
// recording (nothing is created while a capture is open).
template <typename S, typename M>
static hipError_t run_beside(hipStream_t user, S&& side, M&& main)
{
    auto serial = [&]() {
        const hipError_t e = side(user);
        return e == hipSuccess ? main(user) : e;
    };
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_side_mutex);
    SideStream& st = g_side[dev];
    unsigned long long mine = 0, theirs = 0;
    e = capture_of(user, &mine);
    if (e != hipSuccess) return e;
    if (!st.ready) {
        if (mine != 0) return serial();
        e = hipStreamCreateWithFlags(&st.s, hipStreamNonBlocking);  // default priority
        if (e != hipSuccess) return e;
        e = hipEventCreateWithFlags(&st.fork, hipEventDisableTiming);
        if (e == hipSuccess) {
            e = hipEventCreateWithFlags(&st.join, hipEventDisableTiming);
            if (e != hipSuccess) (void)hipEventDestroy(st.fork);
        }
        if (e != hipSuccess) {  // the next call starts over
            (void)hipStreamDestroy(st.s);
            return e;
        }
        st.ready = true;
    }
    e = capture_of(st.s, &theirs);
    if (e != hipSuccess) return e;
    if (theirs != 0 && theirs != mine) return serial();
    e = hipEventRecord(st.fork, user);
    if (e == hipSuccess) e = hipStreamWaitEvent(st.s, st.fork, 0);
    if (e != hipSuccess) return e;
    // what was forked is joined again, whatever happens in between
    hipError_t first = side(st.s);
    if (first == hipSuccess) first = main(user);
    e = hipEventRecord(st.join, st.s);
    if (e == hipSuccess) e = hipStreamWaitEvent(user, st.join, 0);
    return first == hipSuccess ? e : first;
}

// Beside each other only where the longer tensors take a while: the event calls cost the host 46 us a call (sender and
// receiver 92), which a short chain of kernels does not hide.  Sender and receiver in us, beside / serial, by padded samples in
// longer tensors, with 10 and 100 short ones; calls behind each other, and a call that is waited for:
//   2^17 132 / 94 and 145 / 111;  2^21 135 / 119 and 158 / 133;  2^22 143 / 140 and 165 / 157, waited for 167 / 160 and 183 / 190;
//   2^23 180 / 192 and 182 / 208, waited for 226 / 215 and 238 / 244;  2^24 278 / 290 and 280 / 301, waited for 307 / 310 and
//   326 / 333;  2^26 1010 / 1028 and 1014 / 1039, waited for 1054 / 1056 and 1074 / 1081.
// From 2^24 on (kSideUnits) both gain; below, with up to kFewLong longer tensors, their first kernel is in the short ones' launch (chunk.hip).  Per-kernel timing wants one chain.
template <typename S, typename M>
static hipError_t run_segments(const SegmentPlan& plan, hipStream_t user, S&& side, M&& main)
{
    uint32_t units = 0;
    for (const LongBatch& b : plan.longs) units += b.units;
    if (!plan.shorts.empty() && units >= kSideUnits && !prof::enabled()) return run_beside(user, side, main);
    const hipError_t e = side(user);
    return e == hipSuccess ? main(user) : e;
}

extern "C" {

// the stream header's part of the arguments
static CodecArgs segment_header(const size_t* seg_offsets, int nseg, float theta, int bits, int m)
{
    CodecArgs a{};
    a.bits = bits;
    a.m = m;
    a.hdr_n = seg_offsets[nseg] - seg_offsets[0];
    a.hdr_L = 0;
    a.hdr_C = (uint32_t)nseg;
    a.hdr_k = 0;
    a.hdr_S = 0;
    a.hdr_theta = theta;
    return a;
}

static CodecArgs segment_args(const LongBatch& b, const size_t* seg_offsets, int nseg, float theta, int bits, int m)
{
    CodecArgs a = segment_header(seg_offsets, nseg, theta, bits, m);
    a.C = b.count;
    a.tab = &b;
    return a;
}

int fftsp_compress_segments(const float* d_grad, const size_t* seg_offsets, int nseg, float theta, int bits,
                            void* d_packed, size_t packed_capacity, void* d_workspace, size_t workspace_bytes,
                            fftsp_stream_t stream)
{
    int rc = segments_ok(seg_offsets, nseg);
    if (rc) return rc;
    const int m = mantissa(bits);
    if (!theta_ok(theta) || m < 0) return FFTSP_EINVAL;
    if (!d_grad || !d_packed || !d_workspace || !aligned16(d_grad) || !aligned16(d_packed) || !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (packed_capacity < fftsp_packed_bytes_segments(seg_offsets, nseg, theta, bits)) return FFTSP_ENOSPC;
    if (workspace_bytes < fftsp_workspace_bytes_segments(seg_offsets, nseg, bits)) return FFTSP_EWORKSPACE;
    Tables t;
    if (get_tables(&t) != hipSuccess) return FFTSP_EHIP;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    uint8_t* out = static_cast<uint8_t*>(d_packed);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const SegmentPlan plan = plan_segments(seg_offsets, nseg, theta, bits, true);
    if (plan.shorts.size() == 1 && plan.longs.size() == 1 && tensors_compress_beside(plan.shorts[0].tab, plan.longs[0])) {
        const LongBatch& b = plan.longs[0];
        const Workspace w = make_long_workspace(b);
        CodecArgs hdr = segment_header(seg_offsets, nseg, theta, bits, m);
        hdr.write_header = 1;
        float2 *spec = reinterpret_cast<float2*>(ws + w.spec), *mid = reinterpret_cast<float2*>(ws + w.mid);
        uint32_t* hist = reinterpret_cast<uint32_t*>(ws + w.hist);
        hipError_t pe = launch_tensors_compress_beside(d_grad, plan.shorts[0].tab, plan.shorts[0].pieces, QuantizerArgs{bits, m}, hdr, out,
                                                       out + kStreamHeader, b, mid, reinterpret_cast<uint32_t*>(ws + w.status),
                                                       (uint32_t)((w.hist - w.status) / 4 + b.count * (size_t)kHistBins), t, s);
        if (pe == hipSuccess) pe = launch_rfft_b_long(b, spec, mid, t, hist, s);
        if (pe == hipSuccess)
            pe = launch_encode(reinterpret_cast<float*>(spec), segment_args(b, seg_offsets, nseg, theta, bits, m), out, out + kStreamHeader, ws, w, 1, s);
        return hip_status(pe);
    }
    const hipError_t e = run_segments(
        plan, s,
        [&](hipStream_t st) {
            hipError_t pe = hipSuccess;
            for (size_t i = 0; i < plan.shorts.size() && pe == hipSuccess; ++i) {
                CodecArgs hdr = segment_header(seg_offsets, nseg, theta, bits, m);
                hdr.write_header = i == 0;
                // the longer tensors' kernels clear the control block; without any, the first of these launches does
                pe = launch_tensors_compress(d_grad, plan.shorts[i].tab, plan.shorts[i].pieces, plan.shorts[i].top_logL,
                                             QuantizerArgs{bits, m}, hdr, out, out + kStreamHeader,
                                             i == 0 && plan.longs.empty() ? reinterpret_cast<uint32_t*>(ws) : nullptr, t, st);
            }
            return pe;
        },
        [&](hipStream_t st) {
            hipError_t pe = hipSuccess;
            for (size_t i = 0; i < plan.longs.size() && pe == hipSuccess; ++i) {
                const LongBatch& b = plan.longs[i];
                const Workspace w = make_long_workspace(b);
                CodecArgs a = segment_args(b, seg_offsets, nseg, theta, bits, m);
                a.write_header = i == 0 && plan.shorts.empty();
                float2* spec = reinterpret_cast<float2*>(ws + w.spec);
                pe = launch_rfft_long(d_grad, b, spec, reinterpret_cast<float2*>(ws + w.mid), t, reinterpret_cast<uint32_t*>(ws + w.hist),
                                      reinterpret_cast<uint32_t*>(ws + w.status), (w.hist - w.status) / 4 + b.count * (size_t)kHistBins, st);
                if (pe == hipSuccess) pe = launch_encode(reinterpret_cast<float*>(spec), a, out, out + kStreamHeader, ws, w, 1, st);
            }
            return pe;
        });
    return hip_status(e);
}

int fftsp_decompress_segments(const void* d_packed, size_t packed_bytes, float* d_grad_out, const size_t* seg_offsets,
                              int nseg, float theta, int bits, void* d_workspace, size_t workspace_bytes,
                              fftsp_stream_t stream)
{
    int rc = segments_ok(seg_offsets, nseg);
    if (rc) return rc;
    const int m = mantissa(bits);
    if (!theta_ok(theta) || m < 0) return FFTSP_EINVAL;
    if (!d_grad_out || !d_packed || !d_workspace || !aligned16(d_grad_out) || !aligned16(d_packed) ||
        !aligned16(d_workspace))
        return FFTSP_EINVAL;
    if (packed_bytes < fftsp_packed_bytes_segments(seg_offsets, nseg, theta, bits)) return FFTSP_EFORMAT;
    if (workspace_bytes < fftsp_workspace_bytes_segments(seg_offsets, nseg, bits)) return FFTSP_EWORKSPACE;
    Tables t;
    if (get_tables(&t) != hipSuccess) return FFTSP_EHIP;
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    const uint8_t* in = static_cast<const uint8_t*>(d_packed);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const SegmentPlan plan = plan_segments(seg_offsets, nseg, theta, bits, true);
    const size_t verd = segment_verdicts(plan);
    uint32_t* verdicts = reinterpret_cast<uint32_t*>(ws + verd);
    const StatusNote note = status_note((size_t)nseg, verd);
    if (plan.shorts.size() == 1 && plan.longs.size() == 1 && tensors_decompress_beside(plan.shorts[0].tab, plan.shorts[0].pieces, bits, plan.longs[0])) {
        const LongBatch& b = plan.longs[0];
        CodecArgs hdr = segment_header(seg_offsets, nseg, theta, bits, m);
        hdr.write_header = 1;
        const Workspace w = make_long_workspace(b);
        float2* mid = reinterpret_cast<float2*>(ws + w.mid);
        hipError_t pe = launch_tensors_decompress_beside(in, plan.shorts[0].tab, plan.shorts[0].pieces, QuantizerArgs{bits, m}, hdr, d_grad_out,
                                                         reinterpret_cast<uint32_t*>(ws), note, verdicts, b, mid, ws + w.spec, verdicts + plan.short_count, t, s);
        if (pe == hipSuccess && !short_decode(b)) pe = launch_receive_b_long(in, segment_args(b, seg_offsets, nseg, theta, bits, m), ws + w.spec, mid, t, s);
        if (pe == hipSuccess) pe = launch_inverse_a_long(mid, b, d_grad_out, t, s);
        return hip_status(pe);
    }
    const hipError_t e = run_segments(
        plan, s,
        [&](hipStream_t st) {
            hipError_t pe = hipSuccess;
            for (size_t i = 0; i < plan.shorts.size() && pe == hipSuccess; ++i) {
                CodecArgs hdr = segment_header(seg_offsets, nseg, theta, bits, m);
                hdr.write_header = i == 0;
                pe = launch_tensors_decompress(in, plan.shorts[i].tab, plan.shorts[i].pieces, plan.shorts[i].top_logL,
                                               QuantizerArgs{bits, m}, hdr, d_grad_out, reinterpret_cast<uint32_t*>(ws),
                                               i == 0 ? note : StatusNote{}, 1, verdicts, t, st);
            }
            return pe;
        },
        [&](hipStream_t st) {
            hipError_t pe = hipSuccess;
            size_t done = plan.short_count;
            for (size_t i = 0; i < plan.longs.size() && pe == hipSuccess; ++i) {
                const LongBatch& b = plan.longs[i];
                const Workspace w = make_long_workspace(b);
                const bool leads = i == 0 && plan.shorts.empty();
                const CodecArgs a = segment_args(b, seg_offsets, nseg, theta, bits, m);
                float* spec = reinterpret_cast<float*>(ws + w.spec);
                float2* mid = reinterpret_cast<float2*>(ws + w.mid);
                if (short_decode(b)) {
                    pe = launch_short_decode_long(in, a, mid, t, leads, verdicts + done, reinterpret_cast<uint32_t*>(ws + w.status),
                                                  leads ? &note : nullptr, st);
                    if (pe == hipSuccess) pe = launch_inverse_a_long(mid, b, d_grad_out, t, st);
                } else if (receive_applies(b, bits)) {
                    pe = launch_receive_long(in, a, spec, mid, t, leads, verdicts + done, reinterpret_cast<uint32_t*>(ws + w.status),
                                             leads ? &note : nullptr, st);
                    if (pe == hipSuccess) pe = launch_inverse_a_long(mid, b, d_grad_out, t, st);
                } else {
                    pe = launch_decode(in, in + kStreamHeader, a, spec, ws, w, leads, verdicts + done, leads ? &note : nullptr, st);
                    if (pe == hipSuccess) pe = launch_irfft_long(reinterpret_cast<float2*>(spec), b, d_grad_out, mid, t, st);
                }
                done += b.count;
            }
            return pe;
        });
    return hip_status(e);
}

int fftsp_device_status(const void* d_workspace, int* status_out)
{
    if (!d_workspace || !status_out) return FFTSP_EINVAL;
    if (hipDeviceSynchronize() != hipSuccess) return FFTSP_EHIP;
    uint32_t v[kNoteWord + kNoteWords] = {};
    if (hipMemcpy(v, d_workspace, sizeof(v), hipMemcpyDeviceToHost) != hipSuccess) return FFTSP_EHIP;
    uint32_t worst = v[0];
    if (v[4] == kStatusNoteMagic && v[2] > 0) {  // one verdict per record
        std::vector<uint32_t> verdicts(v[2]);
        const uint64_t offset = v[3] | (uint64_t)v[5] << 32;
        if (hipMemcpy(verdicts.data(), static_cast<const uint8_t*>(d_workspace) + offset, verdicts.size() * 4,
                      hipMemcpyDeviceToHost) != hipSuccess)
            return FFTSP_EHIP;
        worst = std::max(worst, *std::max_element(verdicts.begin(), verdicts.end()));
    }
    *status_out = (int)worst;
    return FFTSP_OK;
}

int fftsp_profile_enable(int on)
{
    prof::enable(on != 0);
    return FFTSP_OK;
}

size_t fftsp_profile_report(char* buf, size_t cap)
{
    const std::string r = prof::report();
    if (buf && cap > 0) {
        const size_t ncopy = r.size() < cap - 1 ? r.size() : cap - 1;
        std::memcpy(buf, r.data(), ncopy);
        buf[ncopy] = 0;
    }
    return r.size() + 1;
}

const char* fftsp_strerror(int status)
{
    switch (status) {
        case FFTSP_OK: return "ok";
        case FFTSP_EINVAL: return "invalid argument";
        case FFTSP_ENOSPC: return "packed buffer too small";
        case FFTSP_EWORKSPACE: return "workspace too small";
        case FFTSP_EUNSUPPORTED: return "unsupported chunk length";
        case FFTSP_EHIP: return "HIP runtime error";
        case FFTSP_EFORMAT: return "packed stream does not match the arguments";
        default: return "unknown status";
    }
}

const char* fftsp_version(void) { return "fftsp 0.1 (gfx950)"; }

}  // extern "C"

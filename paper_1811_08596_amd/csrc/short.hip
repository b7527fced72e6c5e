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

#include <type_traits>

namespace fftsp {
namespace {

// points of a pass A tile, by rows: at least four columns
constexpr int short_log_a(int logn1) { return logn1 <= 9 ? 11 : logn1 + 2; }
constexpr int short_lanes_a(int logn1) { return 1 << (short_log_a(logn1) - 3); }
constexpr int kShortSlots = 8;                // rows and mirrors of a pass B tile, side by side: 64 bytes of a run
constexpr int kShortLogSlots = 3;
constexpr int kDecodeMost = 18;  // log2 of the longest half chunk whose bitmap every workgroup counts for itself (RecordBins)

// ------------------------------------------------------------------ pass A ----
// fft.hip multiplies column c of a group of 8 DC by an anchor looked up for column c mod DC and c / DC further factors, one
// after the other.  A tile here is T columns of one such chain: links link0 .. link0 + T - 1 from the anchor's column on.
template <int LOGN1>
struct ShortColumns {
    static constexpr int LOGT = short_log_a(LOGN1) - LOGN1, T = 1 << LOGT;
    static constexpr int LOGHP = LOGN1 - 1, HP = 1 << LOGHP;              // row pairs
    static constexpr int LOGDC = LOGHP < 9 ? 9 - LOGHP : 0, DC = 1 << LOGDC;  // as 512 lanes of fft.hip
    static constexpr int LOGPARTS = 3 - LOGT;                             // tiles of one chain
    static constexpr int LOGSPLIT = LOGDC + LOGPARTS;                     // tiles of a group of columns
    static_assert(LOGT >= 1 && LOGT <= 3, "tiles are parts of a chain");
    uint32_t anchor, link0;
    __device__ __forceinline__ explicit ShortColumns(uint32_t tile)
    {
        link0 = (tile & ((1u << LOGPARTS) - 1u)) << LOGT;
        anchor = ((tile >> LOGSPLIT) << (3 + LOGDC)) + ((tile >> LOGPARTS) & (DC - 1u));
    }
    __device__ __forceinline__ uint32_t column(uint32_t slot) const { return anchor + ((link0 + slot) << LOGDC); }
};

// One tile of the forward pass A.  mid: the chunk's intermediate.
template <int LOGN1, bool HALF>
__device__ __forceinline__ void fwd_a_short(uint32_t tile, const float* __restrict__ in, const Span& sp, int logM,
                                            typename Cx<HALF>::One* __restrict__ mid, const Tables& tb, float in_scale)
{
    using Cols = ShortColumns<LOGN1>;
    constexpr int NT = short_lanes_a(LOGN1), N1 = 1 << LOGN1, LOGT = Cols::LOGT, T = Cols::T, HP = Cols::HP;
    constexpr int KN = HP > NT ? HP / NT : 1;      // row pairs of a lane
    constexpr int SHARE = HP < NT ? NT / HP : 1;   // lanes of a row pair
    constexpr int NC = T / SHARE;                  // its columns of each
    extern __shared__ float2 smem[];
    float2* d = smem;
    float2* tw = smem + (1 << short_log_a(LOGN1));
    const int tid = threadIdx.x;
    const uint32_t M = 1u << logM, N2 = M >> LOGN1;
    const Cols cols(tile);
    float2 v[8];
    const int slot = tid & (T - 1), j = tid >> LOGT;
    static_assert((NT >> LOGT) == N1 / 8, "a lane's loads are the inputs of a radix-8 butterfly");
    load_pairs(v, in, sp, M, (uint32_t)j * N2 + cols.column((uint32_t)slot), (uint32_t)(N1 / 8) * N2, tb);
    const int sh = 22 - logM;
    float2 cur_a[KN], cur_b[KN], ratio_a[KN], ratio_b[KN];
#pragma unroll
    for (int kk = 0; kk < KN; ++kk) {
        const uint32_t ka = (uint32_t)(tid + kk * NT) & (HP - 1), kb = mirror_row(ka, N1);
        cur_a[kk] = twiddle(tb, (cols.anchor * ka) << sh);
        cur_b[kk] = twiddle(tb, (cols.anchor * kb) << sh);
        ratio_a[kk] = twiddle(tb, (ka << Cols::LOGDC) << sh);
        ratio_b[kk] = twiddle(tb, (kb << Cols::LOGDC) << sh);
        if constexpr (HALF) {  // see fft.hip
            cur_a[kk] = make_float2(cur_a[kk].x * in_scale, cur_a[kk].y * in_scale);
            cur_b[kk] = make_float2(cur_b[kk].x * in_scale, cur_b[kk].y * in_scale);
        }
    }
    load_stage_twiddles<LOGN1, NT>(tw, tb, tid);
    bf8<false>(v);
#pragma unroll
    for (int t = 0; t < 8; ++t) d[sw_idx<LOGT>(8 * j + t, slot)] = v[t];
    __syncthreads();
    const uint32_t slot0 = SHARE > 1 ? (uint32_t)(tid >> Cols::LOGHP) * NC : 0u;  // this lane's first column
    for (uint32_t i = 0; i < cols.link0 + slot0; ++i)
#pragma unroll
        for (int kk = 0; kk < KN; ++kk) {
            cur_a[kk] = cmul(cur_a[kk], ratio_a[kk]);
            cur_b[kk] = cmul(cur_b[kk], ratio_b[kk]);
        }
    run_fft<LOGN1, LOGT, NT, false, 3>(d, tw, tid);
    typename Cx<HALF>::Two* out = reinterpret_cast<typename Cx<HALF>::Two*>(mid);
#pragma unroll
    for (int kk = 0; kk < KN; ++kk) {
        const uint32_t ka = (uint32_t)(tid + kk * NT) & (HP - 1), kb = mirror_row(ka, N1);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const uint32_t s = slot0 + (uint32_t)i;
            const float2 va = cmul(d[sw_idx<LOGT>((int)ka, (int)s)], cur_a[kk]);
            const float2 vb = cmul(d[sw_idx<LOGT>((int)kb, (int)s)], cur_b[kk]);
            out[cols.column(s) * (uint32_t)HP + ka] = cx_store<HALF>(join(va, vb));
            cur_a[kk] = cmul(cur_a[kk], ratio_a[kk]);
            cur_b[kk] = cmul(cur_b[kk], ratio_b[kk]);
        }
    }
}

// One tile of the inverse pass A: T adjacent columns.
template <int LOGN1, bool HALF>
__device__ __forceinline__ void inv_a_short(uint32_t tile, const typename Cx<HALF>::One* __restrict__ mid, int logM,
                                            float* __restrict__ out, const Span& sp, const Tables& tb, bool quads_ok, float gain)
{
    constexpr int NT = short_lanes_a(LOGN1), N1 = 1 << LOGN1, LOGT = short_log_a(LOGN1) - LOGN1, T = 1 << LOGT, HP = N1 / 2, LOGHP = LOGN1 - 1;
    extern __shared__ float2 smem[];
    float2* d = smem;
    float2* tw = smem + (1 << short_log_a(LOGN1));
    const int tid = threadIdx.x;
    const uint32_t M = 1u << logM, N2 = M >> LOGN1, col0 = tile << LOGT;
    const typename Cx<HALF>::Two* src = reinterpret_cast<const typename Cx<HALF>::Two*>(mid);
    constexpr int PIECES = (HP * T) / NT;  // 16 bytes each
    static_assert(PIECES == 4, "eight points a lane");
    typename Cx<HALF>::Two r[PIECES];
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
        const int w = tid + q * NT, kp = w & (HP - 1), col = w >> LOGHP;
        r[q] = src[(col0 + (uint32_t)col) * HP + kp];
    }
    load_stage_twiddles<LOGN1, NT>(tw, tb, tid);
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
        const int w = tid + q * NT, kp = w & (HP - 1), col = w >> LOGHP;
        const float4 rq = cx_load(r[q]);
        d[sw_idx<LOGT>(kp, col)] = lo2(rq);
        d[sw_idx<LOGT>((int)mirror_row((uint32_t)kp, N1), col)] = hi2(rq);
    }
    __syncthreads();
    run_fft<LOGN1, LOGT, NT, true, 0>(d, tw, tid);
    const float scale = gain * (1.0f / (float)(2u * M));
    const size_t left = sp.limit > sp.first ? sp.limit - sp.first : 0;
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
        const int w = tid + q * NT, bp = w & (T / 2 - 1), n1 = w >> (LOGT - 1);
        const uint32_t i = (uint32_t)n1 * (N2 >> 1) + (col0 >> 1) + (uint32_t)bp;  // piece of four samples
        const float4 v = lds_load2<LOGT>(d, n1, 2 * bp);
        const float4 s = make_float4(v.x * scale, v.y * scale, v.z * scale, v.w * scale);
        if (quads_ok && 4 * (size_t)i + 4 <= left) {
            reinterpret_cast<float4*>(out + sp.first)[i] = s;
        } else {
            store_pair(out, sp.first + 4 * (size_t)i, sp.limit, lo2(s));
            store_pair(out, sp.first + 4 * (size_t)i + 2, sp.limit, hi2(s));
        }
    }
}

// ------------------------------------------------------------------ pass B ----
// A tile is kShortSlots slots (four rows and their mirrors) of N2 points, a lane one slot.
template <int LOGN2, bool CODEC, bool HALF>
__device__ __forceinline__ void fwd_b_short(uint32_t tile, const typename Cx<HALF>::One* __restrict__ mid, int logM,
                                            typename Cx<HALF>::One* __restrict__ spec, const Tables& tb,
                                            uint32_t* __restrict__ hist, float mid_scale)
{
    using One = typename Cx<HALF>::One;
    constexpr int N2 = 1 << LOGN2, NT = N2, DK = N2 / 8, LOGT = kShortLogSlots;
    extern __shared__ float2 smem[];
    float2* d = smem;
    float2* tw = smem + (N2 << LOGT);
    uint32_t* h16 = reinterpret_cast<uint32_t*>(tw + N2);
    const int tid = threadIdx.x, logN1 = logM - LOGN2;
    const uint32_t M = 1u << logM, N1 = 1u << logN1;
    const int slot = tid & (kShortSlots - 1), kq0 = tid >> LOGT, side = slot & 1;
    const uint32_t place = tile * kShortSlots + (uint32_t)slot, pp = place >> 1, k = side ? mirror_row(pp, N1) : pp;
    One raw[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) raw[q] = mid[((uint32_t)(kq0 + q * DK) << logN1) + place];
    const float2 base = twiddle(tb, (k + ((uint32_t)kq0 << logN1)) << (21 - logM));
    load_stage_twiddles<LOGN2, NT>(tw, tb, tid);
    __shared__ uint32_t range[2];  // highest bucket and the lowest one's complement
    if (CODEC && tid < 2) range[tid] = 0u;
    if (CODEC)
        for (int i = 4 * tid; i < kHistLdsWords; i += 4 * NT) *reinterpret_cast<uint4*>(h16 + i) = make_uint4(0u, 0u, 0u, 0u);
    float2 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = cx_load(raw[q]);
    bf8<false>(v);
#pragma unroll
    for (int t = 0; t < 8; ++t) d[sw_idx<LOGT>(8 * kq0 + t, slot)] = v[t];
    __syncthreads();
    run_fft<LOGN2, LOGT, NT, false, 3>(d, tw, tid);
    const float unlift = HALF ? mid_scale : 1.f, half = 0.5f * unlift;
    uint32_t most = 0, least = kHistBins - 1;  // buckets of this lane's keys
    auto count = [&](float2 x) __attribute__((always_inline)) {
        const uint32_t b = fft_key_of(x) >> kKeyShift;
        most = b > most ? b : most;
        least = b < least ? b : least;
        atomicAdd(&h16[b >> 1], 1u << ((b & 1u) * 16u));
    };
    const bool self = pp == 0;  // rows 0 and N1/2 are their own mirrors
    float2 a[8], p[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int k2 = kq0 + q * DK, back = N2 - 1 - k2;
        const int row = self && side == 0 ? (N2 - k2) & (N2 - 1) : back, other = self ? slot : slot ^ 1;
        a[q] = d[sw_idx<LOGT>(k2, slot)];
        p[q] = d[sw_idx<LOGT>(row, other)];
    }
    const bool dc = self && side == 0 && kq0 == 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int k2 = kq0 + q * DK;
        float2 x = split_fwd(a[q], p[q], cmul(base, make_float2(kW32re[2 * q], kW32im[2 * q])), half);
        if (q == 0 && dc) {  // bin 0 and the Nyquist bin come from Z[0] alone
            x = make_float2((a[0].x + a[0].y) * unlift, 0.f);
            const One last = cx_store<HALF>(make_float2((a[0].x - a[0].y) * unlift, 0.f));
            spec[M] = last;
            if (CODEC) count(cx_load(last));
        }
        if constexpr (CODEC) {
            const One st = cx_store<HALF>(x);
            spec[((uint32_t)k2 << logN1) + place] = st;
            count(cx_load(st));
        } else {
            spec[((uint32_t)k2 << logN1) + k] = x;
        }
    }
    if constexpr (CODEC) {
        // only the stretch of buckets that the tile's keys lie in; neighbouring lanes add to neighbouring counters, which are
        // one access (eight counters to a lane: one chunk of 2^16 10 us instead of 5)
        const uint32_t top = wave_max(most), bottom = ~wave_max(~least);
        if ((tid & 63) == 0) {
            atomicMax(&range[0], top);
            atomicMax(&range[1], ~bottom);
        }
        __syncthreads();
        const uint32_t end = range[0] + 1u;
        const uint16_t* n16 = reinterpret_cast<const uint16_t*>(h16);
        for (uint32_t i = ~range[1] + (uint32_t)tid; i < end; i += NT) {
            const uint32_t n = n16[i];
            if (n) atomicAdd(&hist[i], n);
        }
    }
}

// Where the inverse pass B finds a chunk's bins.
// Spectrum: a buffer in paired or in natural order.
template <bool PAIR, bool HALF>
struct SpectrumBins {
    static constexpr size_t kLds = 0;
    const typename Cx<HALF>::One* spec;
    // x[q]: bin k of run k2 = kq0 + q * DK, last: the Nyquist bin
    template <int LOGN2>
    __device__ __forceinline__ void load(float2 (&x)[8], float2& last, uint32_t place, uint32_t k, int kq0, int logM, float2*, int) const
    {
        constexpr int DK = (1 << LOGN2) / 8;
        typename Cx<HALF>::One raw[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) raw[q] = spec[((uint32_t)(kq0 + q * DK) << (logM - LOGN2)) + (PAIR ? place : k)];
        last = cx_load(spec[1u << logM]);
#pragma unroll
        for (int q = 0; q < 8; ++q) x[q] = cx_load(raw[q]);
    }
};
// Record: the codes of the bins themselves, so that there is no launch that decodes before this one, and no spectrum.  Every
// workgroup counts the chunk's bitmap into a table of its words and the set bits before them (in the LDS that the transform
// will use), and a lane picks the codes of its bins out of memory.
struct RecordArgs {
    uint32_t k, W, S, word3;
    int bits, m;
};
template <bool HALF>
struct RecordBins {
    const uint8_t* record;
    const uint8_t* stream;
    RecordArgs a;
    uint32_t* verdict;  // not null: this workgroup leaves the record's verdict
    bool first;         // the record is its stream's first
    const HeaderInfo& hdr;
    // entry i of the table; one in nine is left out so that lanes eight entries apart use different banks
    static __device__ __forceinline__ uint32_t place_of(uint32_t i) { return i + (i >> 3); }
    template <int LOGN2>
    __device__ __forceinline__ void load(float2 (&x)[8], float2& last, uint32_t, uint32_t k, int kq0, int logM, float2* lds, int tid) const
    {
        constexpr int NT = 1 << LOGN2, DK = NT / 8, MOST = 2 * LOGN2 + 1 < kDecodeMost ? 2 * LOGN2 + 1 : kDecodeMost;
        constexpr int QUADS = 1 << (MOST - LOGN2 - 7);  // of the longest such half chunk
        __shared__ uint32_t before[NT / 64];
        uint2* table = reinterpret_cast<uint2*>(lds);
        const uint32_t* rec = reinterpret_cast<const uint32_t*>(record);
        const int logN1 = logM - LOGN2, quads = 1 << (logN1 - 7);  // a lane's words, in fours
        const uint4* words = reinterpret_cast<const uint4*>(rec + 4) + (uint32_t)tid * (uint32_t)quads;
        uint4 w[QUADS];
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < QUADS; ++i) w[i] = i < quads ? words[i] : make_uint4(0u, 0u, 0u, 0u);
        const uint32_t end = rec[4 + (1u << (logM - 5))] & 1u;  // the Nyquist bin has the last word to itself
        const uint32_t pbase = rec[0];
#pragma unroll
        for (int i = 0; i < QUADS; ++i) sum += (uint32_t)(__popc(w[i].x) + __popc(w[i].y) + __popc(w[i].z) + __popc(w[i].w));
        const uint32_t incl = wave_scan_incl(sum);
        if ((tid & 63) == 63) before[tid >> 6] = incl;
        __syncthreads();
        uint32_t run = incl - sum, all = 0;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) {
            run += i < (tid >> 6) ? before[i] : 0u;
            all += before[i];
        }
#pragma unroll
        for (int i = 0; i < QUADS; ++i) {
            if (i >= quads) break;
            const uint32_t at = 4u * ((uint32_t)tid * (uint32_t)quads + (uint32_t)i), v[4] = {w[i].x, w[i].y, w[i].z, w[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                table[place_of(at + (uint32_t)j)] = make_uint2(v[j], run);
                run += (uint32_t)__popc(v[j]);
            }
        }
        if (verdict && tid == 0) *verdict = record_verdict(record, stream, first, all + (uint32_t)__popc(rec[4 + (1u << (logM - 5))]), a.k, a.word3, hdr);
        __syncthreads();
        const uint32_t* codes = rec + 4 + a.W;
        const int final = a.k ? last_code_word(a.S, a.W) : 0;  // a record with a kept bin has one
        const uint32_t width = 2u * (uint32_t)a.bits;
        const uint32_t base = (pbase - 1u) << (23 - a.m);
        uint32_t rank[9], c0[9], c1[9];
        bool on[9];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t bin = k + ((uint32_t)(kq0 + q * DK) << logN1);
            const uint2 e = table[place_of(bin >> 5)];
            on[q] = (e.x >> (bin & 31u)) & 1u;
            rank[q] = e.y + (uint32_t)__popc(e.x & ((1u << (bin & 31u)) - 1u));
        }
        on[8] = end != 0;
        rank[8] = all;
        // a record without kept bins has no code words; a corrupt bitmap's ranks must not point outside the record
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const int i = on[q] ? code_word(width * rank[q], final) : 0;
            const uint32_t* p = a.k ? codes : rec;
            c0[q] = p[i];
            c1[q] = p[word_after(i, final)];
        }
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            uint32_t re, im;
            if (a.bits == 32) {
                re = on[q] ? c0[q] : 0u;
                im = on[q] ? c1[q] : 0u;
            } else {
                const uint32_t raw = on[q] ? __builtin_amdgcn_alignbit(c1[q], c0[q], width * rank[q]) : 0u;
                re = dequantize_field(raw, 0u, (uint32_t)a.bits, base, 23 - a.m);
                im = dequantize_field(raw, (uint32_t)a.bits, (uint32_t)a.bits, base, 23 - a.m);
            }
            const float2 z = cx_load(cx_store<HALF>(make_float2(__uint_as_float(re), __uint_as_float(im))));
            if (q < 8)
                x[q] = z;
            else
                last = z;
        }
        __syncthreads();
    }
};

template <int LOGN2, bool HALF, typename Bins>
__device__ __forceinline__ void inv_b_short(uint32_t tile, const Bins& bins, int logM, typename Cx<HALF>::One* __restrict__ mid,
                                            const Tables& tb, float mid_scale)
{
    constexpr int N2 = 1 << LOGN2, NT = N2, DK = N2 / 8, LOGT = kShortLogSlots;
    extern __shared__ float2 smem[];
    float2* d = smem;
    float2* tw = smem + (N2 << LOGT);
    const int tid = threadIdx.x, logN1 = logM - LOGN2;
    const uint32_t N1 = 1u << logN1;
    const int slot = tid & (kShortSlots - 1), kq0 = tid >> LOGT, side = slot & 1;
    const uint32_t place = tile * kShortSlots + (uint32_t)slot, pp = place >> 1, k = side ? mirror_row(pp, N1) : pp;
    const bool self = pp == 0, dc = self && side == 0 && kq0 == 0;
    float2 x[8], p[8], last;
    bins.template load<LOGN2>(x, last, place, k, kq0, logM, d, tid);
    const float2 base = twiddle(tb, (k + ((uint32_t)kq0 << logN1)) << (21 - logM));
    const int sh = 22 - logM;
    const float2 ratio = twiddle(tb, ((uint32_t)DK * k) << sh);
    float2 cur = twiddle(tb, ((uint32_t)kq0 * k) << sh);
    if constexpr (HALF) cur = make_float2(cur.x * mid_scale, cur.y * mid_scale);
    load_stage_twiddles<LOGN2, NT>(tw, tb, tid);
#pragma unroll
    for (int q = 0; q < 8; ++q) d[sw_idx<LOGT>(kq0 + q * DK, slot)] = x[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int k2 = kq0 + q * DK, back = N2 - 1 - k2;
        const int row = self && side == 0 ? (N2 - k2) & (N2 - 1) : back, other = self ? slot : slot ^ 1;
        p[q] = d[sw_idx<LOGT>(row, other)];
    }
    if (dc) {  // imaginary parts of the DC and Nyquist bins are ignored
        p[0] = make_float2(last.x, 0.f);
        x[0].y = 0.f;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = split_inv(x[q], p[q], cmul(base, make_float2(kW32re[2 * q], kW32im[2 * q])));
    __syncthreads();
    bf8<true>(x);
#pragma unroll
    for (int t = 0; t < 8; ++t) d[sw_idx<LOGT>(8 * kq0 + t, slot)] = x[t];
    __syncthreads();
    run_fft<LOGN2, LOGT, NT, true, 3>(d, tw, tid);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int n2 = kq0 + q * DK;
        mid[((uint32_t)n2 << logN1) + place] = cx_store<HALF>(cmulc(d[sw_idx<LOGT>(n2, slot)], cur));
        cur = cmul(cur, ratio);
    }
}

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
                                                          float* __restrict__ out, size_t n, Tables tb, int aligned, float gain)
{
    const int log_tiles = logM - short_log_a(LOGN1);
    const uint32_t place = beside<2>(), c = place >> log_tiles;
    inv_a_short<LOGN1, HALF>(place & ((1u << log_tiles) - 1u), mid + ((size_t)c << logM), logM, out,
                             chunk_span(0, n, c, (size_t)2 << logM), tb, (aligned & 2) != 0, gain);
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
constexpr int short_columns(int logM) { return (logM + 1) / 2; }
constexpr int short_rows(int logM) { return logM / 2; }
constexpr int kShortMostA = short_lanes_a(10);
__global__ __launch_bounds__(kShortMostA) void k_fwd_a_long_short(const float* __restrict__ in, float2* __restrict__ mid, Tables tb,
                                                               uint32_t* __restrict__ zero_ptr, uint32_t zero_words, LongTable tab,
                                                               LongStarts at)
{
    clear_words(zero_ptr, zero_words, (int)blockDim.x);
    const LongShare share = long_share(at);
    const LongTensor& x = tab.t[share.tensor];
    const Span sp = chunk_span((size_t)x.goff, x.glen, 0, 0);
    float2* to = mid + long_mid(x);
    if (threadIdx.x >= (uint32_t)short_lanes_a(short_columns(x.logM))) return;
    switch (short_columns(x.logM)) {
        case 8: return fwd_a_short<8, false>(share.blk, in, sp, x.logM, to, tb, 1.0f);
        case 9: return fwd_a_short<9, false>(share.blk, in, sp, x.logM, to, tb, 1.0f);
        default: return fwd_a_short<10, false>(share.blk, in, sp, x.logM, to, tb, 1.0f);
    }
}
__global__ __launch_bounds__(kShortMostA) void k_inv_a_long_short(const float2* __restrict__ mid, float* __restrict__ out, Tables tb, int aligned,
                                                               LongTable tab, LongStarts at)
{
    const LongShare share = long_share(at);
    const LongTensor& x = tab.t[share.tensor];
    const Span sp = chunk_span((size_t)x.goff, x.glen, 0, 0);
    const bool quads = (aligned & 2) && (sp.first & 3u) == 0;
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
    const RecordArgs a{x.kept, (1u << x.logM) / 32u + 1u, x.stride, 2u << x.logM, bits, m};
    const RecordBins<false> bins{records + x.roff, stream, a, share.blk == 0 ? verdicts + share.tensor : nullptr, share.tensor == 0, hdr};
    auto run = [&](auto n2) __attribute__((always_inline)) {
        constexpr int LOGN2 = decltype(n2)::value;
        if (threadIdx.x < (1u << LOGN2)) inv_b_short<LOGN2, false>(share.blk, bins, x.logM, mid + long_mid(x), tb, 1.0f);
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

// ------------------------------------------------------------------ launch ----
template <typename K>
hipError_t short_lds(K kernel, size_t bytes)
{
    if (bytes <= 48 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}
constexpr size_t lds_a(int logn1) { return (((size_t)1 << short_log_a(logn1)) + ((size_t)1 << logn1)) * sizeof(float2); }
constexpr size_t lds_b(int logn2, bool hist)
{
    return ((size_t)(kShortSlots + 1) << logn2) * sizeof(float2) + (hist ? kHistLdsWords * sizeof(uint32_t) : 0);
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
hipError_t launch_a_inv(const float2* mid, int logM, size_t C, float* out, size_t n, Tables t, int aligned, float gain, hipStream_t s)
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

// LDS of the inverse pass B from records: the table of bitmap words (RecordBins), or the tile and its twiddles
constexpr size_t lds_decode(int logM, int logn2)
{
    const size_t words = (size_t)1 << (logM - 5), table = (words + words / 8) * sizeof(uint2);
    return table > lds_b(logn2, false) ? table : lds_b(logn2, false);
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
int alignment(const void* p)
{
    const uintptr_t addr = reinterpret_cast<uintptr_t>(p);
    return ((addr & 7u) == 0 ? 1 : 0) | ((addr & 15u) == 0 ? 2 : 0);
}
template <bool HALF>
hipError_t inv_a_any(const float2* mid, int logM, size_t C, float* out, size_t n, Tables t, float gain, hipStream_t s)
{
    const int aligned = alignment(out);
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
// workgroups of every tensor's share: 2^log(logM) each
template <typename Log>
uint32_t starts_of(const LongBatch& b, LongStarts* at, Log&& log)
{
    uint32_t sum = 0;
    at->first = 0;
    at->count = b.count;
    for (uint32_t i = 0; i < b.count; ++i) {
        at->at[i] = (uint16_t)sum;
        sum += 1u << log((int)b.tab.t[i].logM);
    }
    return sum;
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
    const uint32_t wgs = starts_of(b, &at, [](int log) { return log - short_rows(log) - kShortLogSlots; });
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
    uint32_t wgs = starts_of(b, &at, [](int logM) { return logM - short_log_a(short_columns(logM)); });
    FFTSP_LAUNCH("rfft_pass_a", k_fwd_a_long_short, dim3(wgs), dim3(short_lanes_a(top)), lds_a(top), s, in, mid, t, zero_ptr, zero_words,
                 b.tab, at);
    wgs = starts_of(b, &at, [](int logM) { return logM - short_rows(logM) - kShortLogSlots; });
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
    const uint32_t wgs = starts_of(b, &at, [](int logM) { return logM - short_rows(logM) - kShortLogSlots; });
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
    const uint32_t wgs = starts_of(b, &at, [](int logM) { return logM - short_log_a(short_columns(logM)); });
    FFTSP_LAUNCH("irfft_pass_a", k_inv_a_long_short, dim3(wgs), dim3(short_lanes_a(top)), lds_a(top), s, mid, out, t, alignment(out), b.tab, at);
    return hipGetLastError();
}

}  // namespace fftsp

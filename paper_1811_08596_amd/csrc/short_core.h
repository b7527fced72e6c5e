// Tiles of the short calls' two-pass transforms (short.hip), for every kernel that works on them.
#pragma once
#include "codec_core.h"
#include "fft_core.h"

#include <type_traits>

namespace fftsp {
namespace {

constexpr int short_columns(int logM) { return (logM + 1) / 2; }
constexpr int short_rows(int logM) { return logM / 2; }
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


// ---------------------------------------------------------------- tensors ----
// Tile blk of tensor x.  Lanes a shorter tensor has no use for leave at once (an ended wave takes part in no barrier).
__device__ __forceinline__ void fwd_a_tensor(const LongTensor& x, uint32_t blk, const float* __restrict__ in, float2* __restrict__ mid, const Tables& tb)
{
    const Span sp = chunk_span((size_t)x.goff, x.glen, 0, 0);
    float2* to = mid + long_mid(x);
    if (threadIdx.x >= (uint32_t)short_lanes_a(short_columns(x.logM))) return;
    switch (short_columns(x.logM)) {
        case 8: return fwd_a_short<8, false>(blk, in, sp, x.logM, to, tb, 1.0f);
        case 9: return fwd_a_short<9, false>(blk, in, sp, x.logM, to, tb, 1.0f);
        default: return fwd_a_short<10, false>(blk, in, sp, x.logM, to, tb, 1.0f);
    }
}
// TOP: log2 of the most rows in the launch; verdict: not null where this workgroup leaves the record's
template <int TOP>
__device__ __forceinline__ void decode_tensor(const LongTensor& x, uint32_t blk, const uint8_t* __restrict__ stream, const uint8_t* __restrict__ records,
                                              int bits, int m, const HeaderInfo& hdr, uint32_t* verdict, bool first, float2* __restrict__ mid,
                                              const Tables& tb)
{
    const RecordArgs a{x.kept, (1u << x.logM) / 32u + 1u, x.stride, 2u << x.logM, bits, m};
    const RecordBins<false> bins{records + x.roff, stream, a, verdict, first, hdr};
    auto run = [&](auto n2) __attribute__((always_inline)) {
        constexpr int LOGN2 = decltype(n2)::value;
        if (threadIdx.x < (1u << LOGN2)) inv_b_short<LOGN2, false>(blk, bins, x.logM, mid + long_mid(x), tb, 1.0f);
    };
    const int rows = short_rows(x.logM);
    if (rows == 7) return run(std::integral_constant<int, 7>{});
    if constexpr (TOP >= 8)
        if (rows == 8) return run(std::integral_constant<int, 8>{});
    if constexpr (TOP >= 9)
        if (rows == 9) return run(std::integral_constant<int, 9>{});
}

constexpr size_t lds_a(int logn1) { return (((size_t)1 << short_log_a(logn1)) + ((size_t)1 << logn1)) * sizeof(float2); }
constexpr size_t lds_b(int logn2, bool hist)
{
    return ((size_t)(kShortSlots + 1) << logn2) * sizeof(float2) + (hist ? kHistLdsWords * sizeof(uint32_t) : 0);
}

// LDS of the inverse pass B from records: the table of bitmap words (RecordBins), or the tile and its twiddles
constexpr size_t lds_decode(int logM, int logn2)
{
    const size_t words = (size_t)1 << (logM - 5), table = (words + words / 8) * sizeof(uint2);
    return table > lds_b(logn2, false) ? table : lds_b(logn2, false);
}

}  // namespace
}  // namespace fftsp

// The receiver's first kernels in long calls of two-pass chunk lengths: the inverse pass B takes its bins from the records, so
// that no spectrum is written and read again.
//
// A tile of the pass is 16 slots or more (rows k1 and their mirrors N1 - k1) of N2 points, i.e. eight neighbouring bins of
// either side of every run of N1, or a multiple of that.  The codes of eight neighbouring bins are neighbours in the record, so a
// lane decodes eight of them at a time: it looks up the word of the bitmap and the number of bits before it (one table entry
// for 32 bins, made by k_bitmap_table), fetches a window of the record with two loads, and shifts the codes out of registers.
//
// All tiles of a chunk read the same lines of its record and table, 1.3 MB for a chunk of 2^20.  Workgroups are dealt out to
// the XCDs round-robin, so each XCD gets a stretch of chunks of its own and its workgroups neighbouring tiles of it: the lines come
// over the fabric once and then out of that XCD's L2.
//
// What bounds it: about 100 vector instructions a point (60 of the 116 us below), the two dependent trips to memory before a
// tile's transform, and the barriers in it.  So a lane has eight points and a SIMD eight waves where the tile allows it, and nothing
// is kept for a next tile: a workgroup does one.  (Persistent workgroups of sixteen points a lane that fetched the next tile's entries and
// codes during the transform took 124 to 134 us; a lane that looked up each of its bins alone 187.)
// Measured, 62 M samples in chunks of 2^20, half of the bins kept as 8-bit codes, against counting, decoding and the pass: 6 + 54 + 110
// -> 6 + 116 us; 138 M in chunks of 2^22 15 + 118 + 275 -> 12 + 354; binary16 5 + 33 + 95 -> 6 + 96.
// Several senders' streams are decoded into a spectrum first (codec.hip): eight of them took 444 us this way against 285, since every
// stretch of eight bins is two and a half lines out of L2.
#include "fft_core.h"
#include "codec_core.h"
#include "receive.h"

#include <type_traits>

namespace fftsp {
namespace {

// ------------------------------------------------------------ bitmap table ----
constexpr int kTableLanes = 1024, kTableWaves = kTableLanes / 64;
__host__ __device__ constexpr uint32_t table_stride(int logM) { return (1u << (logM - 5)) + 2u; }  // entries, one to a bitmap word

// Entry i of a record's table: word i of its bitmap and the number of bits set before it.  A workgroup makes kTableWords of them
// and counts the words before its own itself, four loads in flight; the last one of a record leaves the record's verdict.
// (A workgroup per record: sixty records of 2^20 samples 10.8 -> 6.1 us, thirty-three of 2^22 39 -> 12.)
constexpr uint32_t kTableWords = 4 * kTableLanes;
__global__ __launch_bounds__(kTableLanes) void k_bitmap_table(const uint8_t* __restrict__ stream, uint32_t C, size_t S, uint32_t k, HeaderInfo hdr, int logM,
                                                             uint32_t parts, uint2* __restrict__ table, uint32_t* __restrict__ verdicts,
                                                             uint32_t* __restrict__ ctl, StatusNote note)
{
    __shared__ uint32_t own[kTableWaves], earlier[kTableWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the parts of a record share an XCD, and with it the words before theirs (workgroups are dealt out round-robin over the eight)
    const uint32_t y = blockIdx.x >> 3, c = y / parts * 8u + (blockIdx.x & 7u), part = y % parts;
    if (blockIdx.x == 0) clear_control(ctl, note, tid, kTableLanes);
    if (c >= C) return;
    const uint8_t* record = stream + 64 + (size_t)c * S;
    const uint4* quads = reinterpret_cast<const uint4*>(record + 16);
    const uint32_t words = 1u << (logM - 5), at = part * kTableLanes + (uint32_t)tid;  // this lane's four
    auto ones = [](uint4 v) __attribute__((always_inline)) { return (uint32_t)(__popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w)); };
    const bool in = 4u * at < words;
    const uint4 w = in ? quads[at] : make_uint4(0u, 0u, 0u, 0u);
    uint32_t before = 0;
#pragma unroll 4
    for (uint32_t i = 0; i < part; ++i) before += ones(quads[i * kTableLanes + (uint32_t)tid]);
    const uint32_t sum = ones(w), incl = wave_scan_incl(sum);
    before = wave_sum(before);
    if (lane == 63) {
        own[wave] = incl;
        earlier[wave] = before;
    }
    __syncthreads();
    uint32_t run = incl - sum, all = 0;
#pragma unroll
    for (int i = 0; i < kTableWaves; ++i) {
        run += earlier[i] + (i < wave ? own[i] : 0u);
        all += earlier[i] + own[i];
    }
    uint2* out = table + (size_t)c * table_stride(logM);
    if (in) {
        const uint32_t r1 = run + (uint32_t)__popc(w.x), r2 = r1 + (uint32_t)__popc(w.y), r3 = r2 + (uint32_t)__popc(w.z);
        uint4* p = reinterpret_cast<uint4*>(out + 4u * at);  // the stride is even
        p[0] = make_uint4(w.x, run, w.y, r1);
        p[1] = make_uint4(w.z, r2, w.w, r3);
    }
    if (part + 1u == parts && tid == 0) {
        const uint32_t last = reinterpret_cast<const uint32_t*>(quads)[words];  // the Nyquist bin has a word to itself
        *reinterpret_cast<uint4*>(out + words) = make_uint4(last, all, 0u, 0u);
        verdicts[c] = record_verdict(record, stream, c == 0, all + (uint32_t)__popc(last), k, 0u, hdr);
    }
}

// ---------------------------------------------------------- inverse pass B ----
struct RecordShape {
    uint32_t W, S;
    int bits, m;
};
// Eight points a lane and eight waves a SIMD where the tile allows it: what this kernel waits for are its two dependent trips to
// memory and the barriers between the transform's stages, and it moves half the bytes of a transform pass.
template <int LOGN2>
struct Receive {
    static constexpr int N2 = 1 << LOGN2, LOGT = 4, SLOTS = 1 << LOGT;
    static constexpr int U = LOGN2 >= 10 ? 2 : 1, NT = 2 * N2 / U;  // eights of points of a lane
    static constexpr int BINS = SLOTS / 2;                         // neighbouring bins of either side of a run
    static constexpr size_t kLds = ((size_t)(SLOTS + 1) << LOGN2) * sizeof(float2);
};
template <int LOGN2, bool HALF, int WIDEST>
__global__ __launch_bounds__(Receive<LOGN2>::NT) __attribute__((amdgpu_waves_per_eu(8 / Receive<LOGN2>::U, 8 / Receive<LOGN2>::U))) void k_receive_b(
    const uint8_t* __restrict__ records, RecordShape rs, const uint2* __restrict__ table, int logM, typename Cx<HALF>::One* __restrict__ mid,
    Tables tb, uint32_t total, float mid_scale)
{
    using G = Receive<LOGN2>;
    constexpr int N2 = G::N2, NT = G::NT, U = G::U, DK = N2 / 8, LOGT = G::LOGT, SLOTS = G::SLOTS, BINS = G::BINS;
    extern __shared__ float2 smem[];
    float2* d = smem;
    float2* tw = smem + (N2 << LOGT);
    const int tid = threadIdx.x, logN1 = logM - LOGN2, log_tiles = logN1 - LOGT;
    const uint32_t M = 1u << logM, N1 = 1u << logN1;
    // every XCD has a stretch of tiles of its own
    const uint32_t xcd = blockIdx.x & 7u, lo = (uint32_t)((uint64_t)total * xcd >> 3), hi = (uint32_t)((uint64_t)total * (xcd + 1u) >> 3);
    const uint32_t t = lo + (blockIdx.x >> 3);
    if (t >= hi) return;
    const uint32_t c = t >> log_tiles, pp0 = (t & ((1u << log_tiles) - 1u)) * (SLOTS / 2);

    const uint32_t bits = (uint32_t)rs.bits, twoN = 2u * bits;
    const int shift = 23 - rs.m;
    const int final = (int)(rs.S / 4u) - 5 - (int)rs.W;  // a record's last code word
    const uint8_t* record = records + (size_t)c * rs.S;
    const uint32_t* words = reinterpret_cast<const uint32_t*>(record) + 4 + rs.W;
    const uint2* entries = table + (size_t)c * table_stride(logM);
    const uint32_t vbase = (scalar_load(reinterpret_cast<const uint32_t*>(record)) - 1u) << shift;
    auto stored = [](float2 z) __attribute__((always_inline)) { return cx_load(cx_store<HALF>(z)); };  // as a spectrum would hold it

    // A lane's stretch i of bins: run k2, its lower rows (side 0) or the mirrors (side 1).  The latter start at one more than a
    // multiple of eight, so the last bin may be in the bitmap's next word.
    const int k2 = tid & (N2 - 1);
    auto side_of = [&](int i) __attribute__((always_inline)) { return U == 2 ? i : __builtin_amdgcn_readfirstlane(tid >> LOGN2); };
    auto first_of = [&](int i) __attribute__((always_inline)) {  // the stretch's first bin
        return ((uint32_t)k2 << logN1) + (side_of(i) ? N1 - pp0 - (BINS - 1u) : pp0);
    };
    u32x4 entry[U];
#pragma unroll
    for (int i = 0; i < U; ++i) __builtin_memcpy(&entry[i], entries + (first_of(i) >> 5), sizeof(u32x4));
    load_stage_twiddles<LOGN2, NT>(tw, tb, tid);
    Stretch<BINS, WIDEST> o[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const uint32_t at = first_of(i) & 31u, all = (1u << BINS) - 1u;
        // row N1 is the next run's
        o[i].mask = __builtin_amdgcn_alignbit(entry[i][2], entry[i][0], at) & (side_of(i) && pp0 == 0 ? all >> 1 : all);
        o[i].fetch(words, final, (entry[i][1] + (uint32_t)__popc(entry[i][0] & ((1u << at) - 1u))) * twoN);
    }
    // what the lane needs as the transform's: slot and rows kq0 + u * NT / SLOTS + q * N2 / 8
    const int slot = tid & (SLOTS - 1), side = slot & 1;
    const uint32_t pp = pp0 + (uint32_t)(slot >> 1), k = side ? mirror_row(pp, N1) : pp;
    const bool self = pp == 0;
    const int sh = 22 - logM;
    auto kq_of = [&](int u) __attribute__((always_inline)) { return (tid >> LOGT) + u * (NT / SLOTS); };
    float2 base[U], cur[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        base[u] = twiddle(tb, (k + ((uint32_t)kq_of(u) << logN1)) << (21 - logM));
        cur[u] = twiddle(tb, ((uint32_t)kq_of(u) * k) << sh);
        if constexpr (HALF) cur[u] = make_float2(cur[u].x * mid_scale, cur[u].y * mid_scale);
    }
    const float2 ratio = twiddle(tb, ((uint32_t)DK * k) << sh);
#pragma unroll
    for (int i = 0; i < U; ++i)
        o[i].unpack(twoN, bits, shift, vbase, [&](int j, float2 z) __attribute__((always_inline)) {
            d[sw_idx<LOGT>(k2, 2 * (side_of(i) ? BINS - 1 - j : j) + side_of(i))] = stored(z);
        });
    float2 last = make_float2(0.f, 0.f);  // the Nyquist bin
    if (pp0 == 0) {
        // one bin on its own: those outside the stretches
        auto single = [&](uint32_t bin) __attribute__((always_inline)) {
            const uint2 e = entries[bin >> 5];
            const uint32_t bit = (e.y + (uint32_t)__popc(e.x & ((1u << (bin & 31u)) - 1u))) * twoN;
            const int i = (int)(bit >> 5) < final ? (int)(bit >> 5) : final, i1 = i < final ? i + 1 : i;
            const uint32_t raw = (e.x >> (bin & 31u)) & 1u ? __builtin_amdgcn_alignbit(words[i1], words[i], bit) : 0u;
            return stored(make_float2(__uint_as_float(dequantize_field(raw, 0u, bits, vbase, shift)),
                                      __uint_as_float(dequantize_field(raw, bits, bits, vbase, shift))));
        };
        if constexpr (U == 1) __syncthreads();  // the upper lanes have left a zero where row N1/2 goes
        if (tid < N2) d[sw_idx<LOGT>(k2, 1)] = single(((uint32_t)k2 << logN1) + N1 / 2);  // it is its own mirror
        last = single(M);
    }
    __syncthreads();
    // from here on as in fft.hip's inverse pass B
    float2 x[U][8], p[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int r = kq_of(u) + q * DK, back = N2 - 1 - r;
            const int row = self && side == 0 ? (N2 - r) & (N2 - 1) : back, other = self ? slot : slot ^ 1;
            x[u][q] = d[sw_idx<LOGT>(r, slot)];
            p[u][q] = d[sw_idx<LOGT>(row, other)];
        }
    if (self && side == 0 && kq_of(0) == 0) {  // imaginary parts of the DC and Nyquist bins are ignored
        p[0][0] = make_float2(last.x, 0.f);
        x[0][0].y = 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < 8; ++q)
            x[u][q] = split_inv(x[u][q], p[u][q], cmul(base[u], make_float2(kW32re[2 * q], kW32im[2 * q])));
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        bf8<true>(x[u]);
#pragma unroll
        for (int i = 0; i < 8; ++i) d[sw_idx<LOGT>(8 * kq_of(u) + i, slot)] = x[u][i];
    }
    __syncthreads();
    run_fft<LOGN2, LOGT, NT, true, 3>(d, tw, tid);
    typename Cx<HALF>::One* dst = mid + ((size_t)c << logM) + 2u * pp0 + (uint32_t)slot;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int n2 = kq_of(u) + q * DK;
            dst[(uint32_t)n2 << logN1] = cx_store<HALF>(cmulc(d[sw_idx<LOGT>(n2, slot)], cur[u]));
            cur[u] = cmul(cur[u], ratio);
        }
}

// ------------------------------------------------------------------ launch ----
template <int LOGN2, bool HALF, int WIDEST>
hipError_t receive_b(const uint8_t* records, const CodecArgs& a, int logM, const uint2* table, float2* mid, Tables t, hipStream_t s)
{
    using G = Receive<LOGN2>;
    auto kern = k_receive_b<LOGN2, HALF, WIDEST>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::kLds);
    if (e != hipSuccess) return e;
    const size_t total = a.C << (logM - LOGN2 - G::LOGT);
    const RecordShape rs{(1u << logM) / 32u + 1u, (uint32_t)a.S, a.bits, a.m};
    FFTSP_LAUNCH("irfft_pass_b", kern, dim3((unsigned)(8 * ((total + 7) / 8))), dim3(G::NT), G::kLds, s, records, rs, table, logM,
                 reinterpret_cast<typename Cx<HALF>::One*>(mid), t, (uint32_t)total, HALF ? 1.0f / half_lift(logM) : 1.0f);
    return hipGetLastError();
}
template <int LOGN2>
hipError_t receive_rows(const uint8_t* records, const CodecArgs& a, int logM, const uint2* table, float2* mid, Tables t, hipStream_t s)
{
    if (a.half)
        return a.bits <= 8 ? receive_b<LOGN2, true, 16>(records, a, logM, table, mid, t, s)
                           : receive_b<LOGN2, true, 30>(records, a, logM, table, mid, t, s);
    return a.bits <= 8 ? receive_b<LOGN2, false, 16>(records, a, logM, table, mid, t, s)
                       : receive_b<LOGN2, false, 30>(records, a, logM, table, mid, t, s);
}

}  // namespace

// In tiles of 2^13 points.  Whole receivers in us, decode and inverse pass B / these kernels, nothing of a call in the caches when it
// starts, 8-bit codes of half of the bins (chunks of up to 2^19: short.hip's kernels up to 320 tiles).
//   2^16 724 59.6 / 50.4, 4096 285 / 235;  2^17 4096 284 / 212;  2^18 724 64.6 / 50.6, 4096 288 / 220;  2^19 4096 300 / 238;
//   2^20 64 20.5 / 21.4, 128 25.4 / 23.9, 256 33.8 / 29.7, 1024 85.0 / 67.9, 4096 293 / 235;
//   2^21 128 31.3 / 30.2, 1024 96.0 / 75.8, 4096 308 / 279;  2^22 256 47.6 / 38.0, 1024 106 / 83, 4096 347 / 314
constexpr size_t kReceiveFrom = 65;
bool receive_applies(int logM, size_t C, int bits)
{
    return logM >= 15 && bits <= 15 && (C << (logM - 13)) >= kReceiveFrom && (C << (logM - 11)) <= 0x7fffffffu;
}

hipError_t launch_receive(const uint8_t* stream, const CodecArgs& a, int logM, void* table, float2* mid, Tables t, uint32_t* verdicts,
                          uint32_t* ctl, const StatusNote& note, hipStream_t s)
{
    if (!receive_applies(logM, a.C, a.bits)) return hipErrorInvalidValue;
    const HeaderInfo h{1, a.hdr_n, a.hdr_L, a.hdr_C, (uint32_t)a.bits, (uint32_t)a.m, a.hdr_k, a.hdr_S, a.hdr_theta, 0u, (uint32_t)a.hdr_scale};
    uint2* entries = static_cast<uint2*>(table);
    const uint32_t parts = ((1u << (logM - 5)) + kTableWords - 1u) / kTableWords;
    FFTSP_LAUNCH("bitmap_table", k_bitmap_table, dim3((unsigned)((a.C + 7) / 8 * 8 * parts)), dim3(kTableLanes), 0, s, stream, (uint32_t)a.C, a.S, a.k, h, logM, parts, entries,
                 verdicts, ctl, note);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    switch (logM / 2) {
        case 7: return receive_rows<7>(stream + 64, a, logM, entries, mid, t, s);
        case 8: return receive_rows<8>(stream + 64, a, logM, entries, mid, t, s);
        case 9: return receive_rows<9>(stream + 64, a, logM, entries, mid, t, s);
        case 10: return receive_rows<10>(stream + 64, a, logM, entries, mid, t, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fftsp

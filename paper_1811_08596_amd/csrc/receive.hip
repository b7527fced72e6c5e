// The receiver's first kernels in long calls of two-pass chunk lengths: the inverse pass B takes its bins from the records, so
// that no spectrum is written and read again.
//
// A tile of the pass is 16 slots or more (rows k1 and their mirrors N1 - k1) of N2 points, i.e. eight neighbouring bins of
// either side of every run of N1, or a multiple of that.  The codes of eight neighbouring bins are neighbours in the record, so a
// lane decodes eight of them at a time: it looks up the word of the bitmap and the number of bits before it (one table entry
// for 32 bins, made by k_bitmap_table), fetches a window of the record with two loads, and shifts the codes out of registers.
//
// All tiles of a chunk read the same lines of its record and table: 0.66 MB for a chunk of 2^20 samples, half of its bins kept as 8-bit
// codes.  Workgroups are dealt out to the XCDs round-robin, so each XCD gets a stretch of chunks of its own and its workgroups neighbouring
// tiles of it: the lines come over the fabric once and then out of that XCD's L2.
//
// What bounds receive_pairs: the lines that its lanes fetch, since a lane's run of bins is one of its own in the record and one in the table, 16 to 20
// bytes used of each.  In timing builds of whole steps, 62 M samples in chunks of 2^20 / 138 M in 2^22: without the records' windows -27 / -50 us, with windows at neighbouring
// addresses -22 / -41, without the table's entries -12 / -37, without the transform's stages 0 / -9, without the stores 0 / -26.  Its 80 vector instructions a point
// are hidden: codes' values looked up in LDS, a tenth of them less, changed nothing.  A table in the order of the lanes took 7 and 11 us off this kernel and put 6 and 9 on
// the table's.  What helps is tiles beside each other in a compute unit, whose waits another
// one's work fills.  Launches with enough tiles keep a tile in half of the LDS (receive_pairs), which makes it four tiles a compute unit
// for rows of 2^9 and two for 2^10; in shorter ones, a tile or two a compute unit anyhow, the fewer barriers of receive_tile do better.
// (Persistent workgroups of sixteen points a lane that fetched the next tile's entries and codes during the transform took 124 to 134 us where
// receive_tile took 116; a lane that looked up each of its bins alone 187.)
// Measured, 62 M samples in chunks of 2^20, half of the bins kept as 8-bit codes, against counting, decoding and the pass: 6 + 54 + 110
// -> 8 + 101 us; 138 M in chunks of 2^22 15 + 118 + 275 -> 15 + 249; binary16 5 + 33 + 95 -> 7 + 83.
// Tensors of different lengths (ResNet-50's, 34 M samples with their padding): 7 + 32 + 70 -> 7 + 62 (in launches by row length 34 + 34).
// Several senders' streams are decoded into a spectrum first (codec.hip): eight of them took 444 us this way against 285, since every
// stretch of eight bins is two and a half lines out of L2.
#include "fft_core.h"
#include "codec_core.h"
#include "receive.h"
#include "receive_table.h"

#include <type_traits>

namespace fftsp {
namespace {

// ------------------------------------------------------------ bitmap table ----
__global__ __launch_bounds__(kTableLanes) void k_bitmap_table(const uint8_t* __restrict__ stream, uint32_t C, size_t S, uint32_t k, HeaderInfo hdr, int logM,
                                                             uint2* __restrict__ table, uint32_t* __restrict__ verdicts,
                                                             uint32_t* __restrict__ ctl, StatusNote note)
{
    // the parts of a record share an XCD, and with it the words before theirs (workgroups are dealt out round-robin over the eight)
    const uint32_t parts = table_parts(logM), y = blockIdx.x >> 3, c = y / parts * 8u + (blockIdx.x & 7u);
    if (blockIdx.x == 0) clear_control(ctl, note, threadIdx.x, kTableLanes);
    if (c >= C) return;
    bitmap_part(stream, stream + 64 + (size_t)c * S, c == 0, k, 0u, hdr, logM, y % parts, table + (size_t)c * table_stride(logM), verdicts + c);
}
__global__ __launch_bounds__(kTableLanes) void k_bitmap_table_long(const uint8_t* __restrict__ stream, HeaderInfo hdr, uint2* __restrict__ table,
                                                                  uint32_t* __restrict__ verdicts, uint32_t* __restrict__ ctl, StatusNote note,
                                                                  LongTable tab, LongStarts at)
{
    if (ctl && blockIdx.x == 0) clear_control(ctl, note, threadIdx.x, kTableLanes);
    const LongShare share = long_share(at);
    bitmap_part_of_tensor(stream, tab.t[share.tensor], share, hdr, table, verdicts);
}

// ---------------------------------------------------------- inverse pass B ----
// The kernel of short launches: eight points a lane where the tile allows it.
template <int LOGN2>
struct Receive {
    static constexpr int N2 = 1 << LOGN2, LOGT = 4, SLOTS = 1 << LOGT;
    static constexpr int U = LOGN2 >= 10 ? 2 : 1, NT = 2 * N2 / U;  // eights of points of a lane
    static constexpr int WAVES = 8 / U;  // a SIMD: as many as the LDS leaves (rows of 2^7: see receive_b)
    static constexpr int BINS = SLOTS / 2;                         // neighbouring bins of either side of a run
    static constexpr size_t kLds = ((size_t)(SLOTS + 1) << LOGN2) * sizeof(float2);
};
// A tile of rows and mirrors from pp0 on, by G::NT lanes; mid: the chunk's.  Several tiles of a workgroup run beside each other, each
// in LDS of its own; first: whether row 0 is in one of them.
template <int LOGN2, bool HALF, int WIDEST>
__device__ __forceinline__ void receive_tile(const uint8_t* __restrict__ record, uint32_t W, uint32_t S, int code_bits, int m,
                                             const uint2* __restrict__ entries, int logM, typename Cx<HALF>::One* __restrict__ mid, Tables tb,
                                             uint32_t pp0, bool first, float2* d, int tid, float mid_scale)
{
    using G = Receive<LOGN2>;
    constexpr int N2 = G::N2, NT = G::NT, U = G::U, DK = N2 / 8, LOGT = G::LOGT, SLOTS = G::SLOTS, BINS = G::BINS;
    float2* tw = d + (N2 << LOGT);
    const int logN1 = logM - LOGN2;
    const uint32_t M = 1u << logM, N1 = 1u << logN1;

    const uint32_t bits = (uint32_t)code_bits, twoN = 2u * bits;
    const int shift = 23 - m;
    const int final = last_code_word(S, W);
    const uint32_t* words = reinterpret_cast<const uint32_t*>(record) + 4 + W;
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
    for (int i = 0; i < U; ++i) __builtin_memcpy(&entry[i], reinterpret_cast<const uint8_t*>(entries) + (first_of(i) >> 5) * 8u, sizeof(u32x4));
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
    float2 base[U], cur[U], ratio;
#pragma unroll
    for (int u = 0; u < U; ++u) base[u] = twiddle(tb, (k + ((uint32_t)kq_of(u) << logN1)) << (21 - logM));
    auto outer_twiddles = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            cur[u] = twiddle(tb, ((uint32_t)kq_of(u) * k) << sh);
            if constexpr (HALF) cur[u] = make_float2(cur[u].x * mid_scale, cur[u].y * mid_scale);
        }
        ratio = twiddle(tb, ((uint32_t)DK * k) << sh);
    };
    // with sixteen points a lane the split wants their registers: 138 M samples in chunks of 2^22 354 -> 340 us
    if constexpr (U == 1) outer_twiddles();
#pragma unroll
    for (int i = 0; i < U; ++i)
        o[i].unpack(twoN, bits, shift, vbase, [&](int j, float2 z) __attribute__((always_inline)) {
            d[sw_idx<LOGT>(k2, 2 * (side_of(i) ? BINS - 1 - j : j) + side_of(i))] = stored(z);
        });
    float2 last = make_float2(0.f, 0.f);  // the Nyquist bin
    if (first) {
        if constexpr (U == 1) __syncthreads();  // the upper lanes have left a zero where row N1/2 goes
        // one bin on its own: those outside the stretches
        auto single = [&](uint32_t bin) __attribute__((always_inline)) {
            const uint2 e = entries[bin >> 5];
            const uint32_t bit = (e.y + (uint32_t)__popc(e.x & ((1u << (bin & 31u)) - 1u))) * twoN;
            const int i = code_word(bit, final), i1 = word_after(i, final);
            const uint32_t raw = (e.x >> (bin & 31u)) & 1u ? __builtin_amdgcn_alignbit(words[i1], words[i], bit) : 0u;
            return stored(make_float2(__uint_as_float(dequantize_field(raw, 0u, bits, vbase, shift)),
                                      __uint_as_float(dequantize_field(raw, bits, bits, vbase, shift))));
        };
        if (pp0 == 0) {
            if (tid < N2) d[sw_idx<LOGT>(k2, 1)] = single(((uint32_t)k2 << logN1) + N1 / 2);  // it is its own mirror
            last = single(M);
        }
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
    if constexpr (U > 1) outer_twiddles();
    __syncthreads();
    // one base for all lanes and 32-bit offsets: a chunk is 16 MB at most
    auto store = [&](uint32_t i, typename Cx<HALF>::One z) __attribute__((always_inline)) {
        *reinterpret_cast<typename Cx<HALF>::One*>(reinterpret_cast<uint8_t*>(mid) + i * (uint32_t)sizeof(z)) = z;
    };
    const uint32_t column = 2u * pp0 + (uint32_t)slot;
    auto out = [&](int u, int q, float2 z) __attribute__((always_inline)) {
        store(((uint32_t)(kq_of(u) + q * DK) << logN1) + column, cx_store<HALF>(cmulc(z, cur[u])));
        cur[u] = cmul(cur[u], ratio);
    };
    if constexpr (LOGN2 > 7) {
        // A last stage of radix 8 leaves every lane what it stores, so a trip through LDS and two barriers are saved: long launches of it, chunks of
        // 2^22 344 -> 317 us, of 2^20 in binary16 101 -> 94.
        run_fft_put<LOGN2, LOGT, NT, true, 3>(d, tw, tid, out);
    } else {
        run_fft<LOGN2, LOGT, NT, true, 3>(d, tw, tid);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < 8; ++q) out(u, q, d[sw_idx<LOGT>(kq_of(u) + q * DK, slot)]);
    }
}

// The kernel of long launches: a tile in half of the LDS and half of the lanes, sixteen points each.
//
// What goes through LDS before the split are the codes, a word to a bin, [side][run][pair]: a lane writes the eight of a stretch as they lie
// and reads, of a pair of slots, rows that are each other's mirrors, so that every bin is read once and a lane has both of a split's
// inputs.  Those rows are also the inputs of two radix-8 butterflies.  Between the stages real and imaginary parts go through LDS one after
// the other.  The last stage goes to memory from registers.  Same arithmetic as receive_tile, bit for bit.
//
// Eight waves a SIMD (64 registers, none spilled): with six, 62 M samples in chunks of 2^20 104 -> 110 us, binary16 82 -> 86, 40 M in chunks
// of 2^16 58 -> 60.  Outer twiddles fetched before the stages: 104 -> 106, 82 -> 84.
template <int LOGN2, bool HALF, int WIDEST>
__device__ __forceinline__ void receive_pairs(const uint8_t* __restrict__ record, uint32_t W, uint32_t S, int code_bits, int m,
                                              const uint2* __restrict__ entries, int logM, typename Cx<HALF>::One* __restrict__ mid, Tables tb,
                                              uint32_t pp0, bool first, uint32_t* lds, int tid, float mid_scale)
{
    using G = HalfTile<LOGN2>;
    constexpr int N2 = G::N2, NT = G::NT, DK = G::DK, BINS = G::PAIRS;
    float* const d = reinterpret_cast<float*>(lds);
    float2* const tw = reinterpret_cast<float2*>(lds + N2 * G::SLOTS);
    const int logN1 = logM - LOGN2;
    const uint32_t M = 1u << logM, N1 = 1u << logN1;

    const uint32_t bits = (uint32_t)code_bits, twoN = 2u * bits;
    const int shift = 23 - m;
    const int final = last_code_word(S, W);
    const uint32_t* words = reinterpret_cast<const uint32_t*>(record) + 4 + W;
    uint32_t vbase = (scalar_load(reinterpret_cast<const uint32_t*>(record)) - 1u) << shift;

    // A lane's two stretches of bins: run tid, its lower rows and the mirrors.  The latter start at one more than a multiple of
    // eight, so the last bin may be in the bitmap's next word.
    auto first_of = [&](int i) __attribute__((always_inline)) {  // the stretch's first bin
        return ((uint32_t)tid << logN1) + (i ? N1 - pp0 - (BINS - 1u) : pp0);
    };
    u32x4 entry[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) __builtin_memcpy(&entry[i], reinterpret_cast<const uint8_t*>(entries) + (first_of(i) >> 5) * 8u, sizeof(u32x4));
    load_stage_twiddles<LOGN2, NT>(tw, tb, tid);
    Stretch<BINS, WIDEST> o[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t at = first_of(i) & 31u, all = (1u << BINS) - 1u;
        // row N1 is the next run's
        o[i].mask = __builtin_amdgcn_alignbit(entry[i][2], entry[i][0], at) & (i && pp0 == 0 ? all >> 1 : all);
        o[i].fetch(words, final, (entry[i][1] + (uint32_t)__popc(entry[i][0] & ((1u << at) - 1u))) * twoN);
    }
    const int j = tid & (BINS - 1);
    const MirroredRows<LOGN2> rows(pp0 + (uint32_t)j, tid >> 3);
    float2 base[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t pp = pp0 + (uint32_t)j, k = rows.upper(i) ? mirror_row(pp, N1) : pp;
        base[i] = twiddle(tb, (k + ((uint32_t)rows.at(i) << logN1)) << (21 - logM));
    }
    // codes[side][run][pair]
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        uint32_t code[BINS];
        o[i].unpack_codes(twoN, [&](int b, uint32_t raw) __attribute__((always_inline)) { code[i ? BINS - 1 - b : b] = raw; });
        uint4* to = reinterpret_cast<uint4*>(lds + (i * N2 + tid) * BINS);
        to[0] = make_uint4(code[0], code[1], code[2], code[3]);
        to[1] = make_uint4(code[4], code[5], code[6], code[7]);
    }
    asm("" : "+v"(vbase));  // in a vector register, so that it is the addend of a shift-and-add
    auto value = [&](uint32_t raw) __attribute__((always_inline)) {  // as a spectrum would hold it
        return cx_load(cx_store<HALF>(make_float2(__uint_as_float(dequantize_field(raw, 0u, bits, vbase, shift)),
                                                  __uint_as_float(dequantize_field(raw, bits, bits, vbase, shift)))));
    };
    float last = 0.f;  // the Nyquist bin
    if (first) {
        // one bin on its own: those outside the stretches
        auto single = [&](uint32_t bin) __attribute__((always_inline)) {
            const uint2 e = entries[bin >> 5];
            const uint32_t bit = (e.y + (uint32_t)__popc(e.x & ((1u << (bin & 31u)) - 1u))) * twoN;
            const int i = code_word(bit, final), i1 = word_after(i, final);
            return (e.x >> (bin & 31u)) & 1u ? __builtin_amdgcn_alignbit(words[i1], words[i], bit) : 0u;
        };
        if (pp0 == 0) {
            lds[(N2 + tid) * BINS] = single(((uint32_t)tid << logN1) + N1 / 2);  // it is its own mirror
            last = value(single(M)).x;
        }
    }
    __syncthreads();
    float2 v[16];
    {
        const uint32_t *a = lds + (rows.upper(0) * N2 + rows.at(0)) * BINS + j, *b = lds + (rows.upper(1) * N2 + rows.at(1)) * BINS + j;
        const bool alone = rows.alone;
        auto turned = [&](int i, int q) __attribute__((always_inline)) { return cmul(base[i], make_float2(kW32re[2 * q], kW32im[2 * q])); };
        if (first) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                asm volatile("" ::: "memory");  // one after the other: all at once take more registers than there are
                float2 x = value(a[q * DK * BINS]), y = value((alone ? a : b)[(alone ? (8 - q) & 7 : 7 - q) * DK * BINS]);
                if (q == 0 && alone) {  // imaginary parts of the DC and Nyquist bins are ignored
                    x.y = 0.f;
                    y = make_float2(last, 0.f);
                }
                v[q] = split_inv(x, y, turned(0, q));
                v[15 - q] = split_inv(value(b[(7 - q) * DK * BINS]), value((alone ? b : a)[q * DK * BINS]), turned(1, 7 - q));
            }
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float2 x = value(a[q * DK * BINS]), y = value(b[(7 - q) * DK * BINS]);
                v[q] = split_inv(x, y, turned(0, q));
                v[15 - q] = split_inv(y, x, turned(1, 7 - q));
            }
        }
    }
    bf8<true>(v);
    bf8<true>(v + 8);
    const int slot = tid & 15;
    // What the lane stores: two chains of eight rows of its slot, an eighth of the rows apart, with their twiddles.
    constexpr int RHO = 1 << G::LAST, CHAINS = RHO / 8;
    const uint32_t column = 2u * pp0 + (uint32_t)slot, k = slot & 1 ? mirror_row(pp0 + (uint32_t)(slot >> 1), N1) : pp0 + (uint32_t)(slot >> 1);
    auto first_row = [&](int g) __attribute__((always_inline)) { return G::row_of(tid, g / CHAINS) + g % CHAINS * (N2 / RHO); };
    const int sh = 22 - logM;
    float2 cur[2], ratio;
    auto outer_twiddles = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            cur[g] = twiddle(tb, ((uint32_t)first_row(g) * k) << sh);
            if constexpr (HALF) cur[g] = make_float2(cur[g].x * mid_scale, cur[g].y * mid_scale);
        }
        ratio = twiddle(tb, ((uint32_t)DK * k) << sh);
    };
    auto row_of = [&](int q) __attribute__((always_inline)) { return G::row_of(tid, q); };
    G::exchange(
        d, v, [&](int n) __attribute__((always_inline)) { return G::first_output(rows.at(n >> 3), n & 7, rows.upper(n >> 3) * BINS + j); },
        [&](int n) __attribute__((always_inline)) { return G::template input<G::RL2>(tid, n); });
    G::template stage<true, 3, G::RL2>(v, tw, row_of);
    if constexpr (G::RL3 > 0) {
        G::exchange(
            d, v, [&](int n) __attribute__((always_inline)) { return G::second_output(tid, n); },
            [&](int n) __attribute__((always_inline)) { return G::template input<G::LAST>(tid, n); });
        G::template stage<true, 3 + G::RL2, G::LAST>(v, tw, row_of);
    }
    outer_twiddles();
    // one base for all lanes and 32-bit offsets: a chunk is 16 MB at most
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        float2 z = cur[g];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t i = ((uint32_t)(first_row(g) + u * DK) << logN1) + column;
            *reinterpret_cast<typename Cx<HALF>::One*>(reinterpret_cast<uint8_t*>(mid) + i * (uint32_t)sizeof(typename Cx<HALF>::One)) =
                cx_store<HALF>(cmulc(v[g / CHAINS * RHO + g % CHAINS + u * CHAINS], z));
            z = cmul(z, ratio);
        }
    }
}

template <int LOGN2, bool HALF, int WIDEST, int WAVES>
__global__ __launch_bounds__(Receive<LOGN2>::NT) __attribute__((amdgpu_waves_per_eu(WAVES, WAVES))) void k_receive_b(
    const uint8_t* __restrict__ records, uint32_t W, uint32_t S, int bits, int m, const uint2* __restrict__ table, int logM,
    typename Cx<HALF>::One* __restrict__ mid, Tables tb, uint32_t total, float mid_scale)
{
    using G = Receive<LOGN2>;
    extern __shared__ float2 smem[];
    const int log_tiles = logM - LOGN2 - G::LOGT;
    const uint32_t t = in_stretches(total);
    if (t >= total) return;
    const uint32_t c = t >> log_tiles, pp0 = (t & ((1u << log_tiles) - 1u)) * (G::SLOTS / 2);
    receive_tile<LOGN2, HALF, WIDEST>(records + (size_t)c * S, W, S, bits, m, table + (size_t)c * table_stride(logM), logM, mid + ((size_t)c << logM), tb,
                                      pp0, pp0 == 0, smem, threadIdx.x, mid_scale);
}
template <int LOGN2, bool HALF, int WIDEST>
__global__ __launch_bounds__(HalfTile<LOGN2>::NT) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_receive_pairs(
    const uint8_t* __restrict__ records, uint32_t W, uint32_t S, int bits, int m, const uint2* __restrict__ table, int logM,
    typename Cx<HALF>::One* __restrict__ mid, Tables tb, uint32_t total, float mid_scale)
{
    extern __shared__ float2 smem[];
    const int log_tiles = logM - LOGN2 - 4;
    const uint32_t t = in_stretches(total);
    if (t >= total) return;
    const uint32_t c = t >> log_tiles, pp0 = (t & ((1u << log_tiles) - 1u)) * 8u;
    receive_pairs<LOGN2, HALF, WIDEST>(records + (size_t)c * S, W, S, bits, m, table + (size_t)c * table_stride(logM), logM, mid + ((size_t)c << logM), tb,
                                       pp0, pp0 == 0, reinterpret_cast<uint32_t*>(smem), threadIdx.x, mid_scale);
}
// Tensors of different lengths, rows of up to 2^9 (TOP 9: a workgroup of 1024 lanes does one tile of rows of 2^9, two of 2^8 or four of 2^7) or of 2^10
// alone (TOP 10).
template <int TOP, int WIDEST>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(Receive<TOP>::WAVES, Receive<TOP>::WAVES))) void k_receive_b_long(
    const uint8_t* __restrict__ records, int bits, int m, const uint2* __restrict__ table, float2* __restrict__ mid, Tables tb, uint32_t total, uint32_t few,
    LongTable tab, LongStarts at)
{
    static_assert(Receive<TOP>::NT == 1024, "one tile of the longest rows");
    extern __shared__ float2 smem[];
    const uint32_t t = in_stretches(total, few);
    if (t >= total) return;
    const LongShare share = long_share(at, t);
    const LongTensor& x = tab.t[share.tensor];
    auto run = [&](auto n2) __attribute__((always_inline)) {
        constexpr int LOGN2 = decltype(n2)::value, LOGSUB = LOGN2 < TOP ? TOP - LOGN2 : 0;
        using G = Receive<LOGN2>;
        static_assert(G::NT << LOGSUB == 1024, "tiles beside each other");
        const uint32_t sub = LOGSUB ? (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / G::NT) : 0u, pp0 = ((share.blk << LOGSUB) + sub) * (G::SLOTS / 2);
        receive_tile<LOGN2, false, WIDEST>(records + x.roff, (1u << x.logM) / 32u + 1u, x.stride, bits, m, table + long_entries(x, share.tensor), x.logM,
                                           mid + long_mid(x), tb, pp0, share.blk == 0, smem + (size_t)sub * (G::kLds / sizeof(float2)),
                                           threadIdx.x & (G::NT - 1), 1.0f);
    };
    if constexpr (TOP == 9) {
        const int rows = x.logM / 2;
        if (rows == 7) return run(std::integral_constant<int, 7>{});
        if (rows == 8) return run(std::integral_constant<int, 8>{});
    }
    run(std::integral_constant<int, TOP>{});
}

// The same in halves of the LDS, rows of any lengths up to 2^TOP: a tile of rows of 2^TOP, two of half the length, and so on.
template <int TOP, int WIDEST>
__global__ __launch_bounds__(HalfTile<TOP>::NT) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_receive_pairs_long(
    const uint8_t* __restrict__ records, int bits, int m, const uint2* __restrict__ table, float2* __restrict__ mid, Tables tb, uint32_t total, uint32_t few,
    LongTable tab, LongStarts at)
{
    extern __shared__ float2 smem[];
    const uint32_t t = in_stretches(total, few);
    if (t >= total) return;
    const LongShare share = long_share(at, t);
    const LongTensor& x = tab.t[share.tensor];
    auto run = [&](auto n2) __attribute__((always_inline)) {
        constexpr int LOGN2 = decltype(n2)::value, LOGSUB = LOGN2 < TOP ? TOP - LOGN2 : 0;
        using G = HalfTile<LOGN2>;
        const uint32_t sub = LOGSUB ? (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / G::NT) : 0u, pp0 = ((share.blk << LOGSUB) + sub) * 8u;
        receive_pairs<LOGN2, false, WIDEST>(records + x.roff, (1u << x.logM) / 32u + 1u, x.stride, bits, m, table + long_entries(x, share.tensor), x.logM,
                                            mid + long_mid(x), tb, pp0, share.blk == 0, reinterpret_cast<uint32_t*>(smem) + sub * (G::kLds / 4),
                                            threadIdx.x & (G::NT - 1), 1.0f);
    };
    const int rows = x.logM / 2;
    if (rows == 7) return run(std::integral_constant<int, 7>{});
    if (rows == 8) return run(std::integral_constant<int, 8>{});
    if (TOP == 9 || rows == 9) return run(std::integral_constant<int, 9>{});
    if constexpr (TOP == 10) run(std::integral_constant<int, 10>{});
}

// ------------------------------------------------------------------ launch ----
template <int LOGN2, bool HALF, int WIDEST>
hipError_t receive_b(const uint8_t* records, const CodecArgs& a, int logM, const uint2* table, float2* mid, Tables t, hipStream_t s)
{
    const size_t total = a.C << (logM - LOGN2 - 4);
    // Whole receivers in us, receive_tile / receive_pairs, 8-bit codes of 40 %, by tiles; binary16 behind a semicolon:
    //   rows of 2^7 (2^16), receive_tile with eight waves a SIMD, four registers spilled / with six / receive_pairs: 1536 34.6 / 35.2, 2048 36.4 / 37.1 / 37.1; 34.7 / 34.9 /
    //     36.8, 2560 42.2 / 42.5 / 46.0; 41.6 / 42.4 / 45.5, 3072 45.1 / 45.9 / 46.5; 43.7 / 44.8 / 46.9, 3328 48.7 / 45.5 / 47.0; 44.4 / 45.3 / 47.4, 3584 53.0 / 48.9 / 48.3; 45.7 /
    //     46.4 / 48.9, 4096 60.6 / 56.6 / 54.7; 51.2 / 50.1 / 51.4, 4352 65.8 / 61.2 / 58.3; 58.2 / 55.7 / 55.5, 6400 90.7 / 83.8 / 80.1; 76.7 / 72.7 / 70.3;
    //   rows of 2^8 (2^17): 1280 43.6 / 44.9; 42.5 / 45.6, 1920 52.5 / 54.3; 48.5 / 51.9, 2176 59.9 / 59.9; 55.7 / 56.8, 2304 62.1 / 61.0; 56.8 / 57.1, 2560 66.4 / 66.1; 59.9 / 59.3;
    //     (2^18) 1920 52.3 / 54.8; 46.9 / 49.6, 2176 59.4 / 59.5; 52.6 / 53.6, 2304 61.5 / 60.4; 53.9 / 54.0, 2560 65.8 / 65.4; 58.4 / 57.1;
    //   rows of 2^9 (2^19): 256 27.0 / 27.0, 384 36.6 / 35.2; 34.2 / 35.0, 640 43.1 / 43.5; 41.2 / 44.1, 1024 58.0 / 55.3; 51.6 / 53.8, 1088 57.3 / 56.5 (binary16), 1536
    //     82.5 / 77.7; 70.3 / 67.6;  (2^20) 320 36.0 / 35.2; 34.0 / 33.4, 640 45.0 / 44.7; 42.9 / 44.4, 1024 60.0 / 55.7; 55.1 / 55.0, 3840 225 / 210;
    //   rows of 2^10 (2^21): 256 41.2 / 43.6; 39.7 / 42.2, 320 55.8 / 52.8; 54.1 / 52.8, 1024 115.9 / 103.5; 108.3 / 97.8;  (2^22) 256 46.9 / 48.2; 44.1 / 45.3, 384 63.2 / 59.1;
    //     59.8 / 58.2.
    constexpr size_t kPairsFrom = LOGN2 == 7 ? (HALF ? 4224 : 3584) : LOGN2 == 8 ? (HALF ? 2305 : 2177) : LOGN2 == 9 && HALF ? 1025 : 257;
    constexpr size_t kSixWavesFrom = HALF ? 3840 : 2561;  // rows of 2^7
    auto launch = [&](auto kern, unsigned lanes, size_t lds) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        FFTSP_LAUNCH("irfft_pass_b", kern, dim3((unsigned)(8 * ((total + 7) / 8))), dim3(lanes), lds, s, records, (1u << logM) / 32u + 1u, (uint32_t)a.S,
                     a.bits, a.m, table, logM, reinterpret_cast<typename Cx<HALF>::One*>(mid), t, (uint32_t)total, HALF ? 1.0f / half_lift(logM) : 1.0f);
        return hipGetLastError();
    };
    using G = Receive<LOGN2>;
    if (total >= kPairsFrom) return launch(k_receive_pairs<LOGN2, HALF, WIDEST>, HalfTile<LOGN2>::NT, HalfTile<LOGN2>::kLds);
    if constexpr (LOGN2 == 7)
        if (total >= kSixWavesFrom) return launch(k_receive_b<LOGN2, HALF, WIDEST, 6>, G::NT, G::kLds);
    return launch(k_receive_b<LOGN2, HALF, WIDEST, G::WAVES>, G::NT, G::kLds);
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
//   2^16 724 59.6 / 50.4, 4096 284 / 220;  2^17 4096 284 / 212;  2^18 724 64.6 / 50.6, 4096 288 / 220;  2^19 4096 300 / 238;
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
    FFTSP_LAUNCH("bitmap_table", k_bitmap_table, dim3((unsigned)((a.C + 7) / 8 * 8 * table_parts(logM))), dim3(kTableLanes), 0, s, stream, (uint32_t)a.C, a.S,
                 a.k, h, logM, entries, verdicts, ctl, note);
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

// Tensors of different lengths.  Whole receivers of per-tensor calls in us, by tiles, decode and inverse pass B / these kernels, half of the bins as
// 8-bit codes:
//   rows of up to 2^9 alone 128 26.8 / 26.1, 192 31.4 / 29.0, 480 52.7 / 45.2 and 47.5 / 40.7;  of 2^10 alone 128 31.2 / 34.5, 256
//   43.5 / 41.8, 512 62.3 / 50.7;
// both, one launch, sender and receiver, 30 % as 8-bit codes: 180 142.3 / 143.8, 216 145.7 / 147.0, 268 161.3 / 157.0, 292 161.9 / 158.7 and 159.3 / 154.7,
//   320 161.9 / 159.3, 412 172.0 / 165.4, 512 174.0 / 164.1, 616 211.3 / 199.4, 732 221.2 / 208.0, 880 241.2 / 221.0, 944 260.2 / 235.4.
//   Receivers alone by codes, at 256 tiles, 5 / 30 / 90 % as 8-bit codes 42.4 / 38.5, 42.6 / 40.0, 42.5 / 41.6, as 12-bit ones 42.5 / 39.3, - , 42.9 / 42.1, 30 % as 15-bit ones 42.8 /
//   40.6;  at 416 5 and 90 % as 8-bit codes 47.8 / 41.5 and 48.1 / 44.2, as 12-bit ones 48.8 / 42.4 and 50.9 / 44.7.
constexpr size_t kReceiveTallFrom = 192, kReceiveBothFrom = 256;
bool receive_applies(const LongBatch& b, int bits)
{
    auto tall = [&](uint32_t i) { return b.tab.t[i].logM / 2 >= 10; };  // the longest come last
    const size_t tiles = (size_t)b.units << (kLongUnitLog - 13);
    return bits <= 15 && tiles >= (tall(0) ? kReceiveTallFrom : (tall(b.count - 1) ? kReceiveBothFrom : kReceiveFrom));
}

hipError_t launch_receive_long(const uint8_t* stream, const CodecArgs& a, void* table, float2* mid, Tables t, int check_header, uint32_t* verdicts,
                               uint32_t* ctl, const StatusNote* first, hipStream_t s)
{
    const LongBatch& b = *a.tab;
    if (!receive_applies(b, a.bits)) return hipErrorInvalidValue;
    const HeaderInfo h{check_header, a.hdr_n, a.hdr_L, a.hdr_C, (uint32_t)a.bits, (uint32_t)a.m, a.hdr_k, a.hdr_S, a.hdr_theta, 0u, 0u};
    uint2* entries = static_cast<uint2*>(table);
    LongStarts at;
    const uint32_t parts = long_starts(b, 0, b.count, &at, [](int logM) { return table_parts(logM); });
    FFTSP_LAUNCH("bitmap_table", k_bitmap_table_long, dim3(parts), dim3(kTableLanes), 0, s, stream, h, entries, verdicts, first ? ctl : nullptr,
                 first ? *first : StatusNote{}, b.tab, at);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? launch_receive_b_long(stream, a, table, mid, t, s) : e;
}

hipError_t launch_receive_b_long(const uint8_t* stream, const CodecArgs& a, const void* table, float2* mid, Tables t, hipStream_t s)
{
    const LongBatch& b = *a.tab;
    if (!receive_applies(b, a.bits)) return hipErrorInvalidValue;
    const uint2* entries = static_cast<const uint2*>(table);
    LongStarts at;
    hipError_t e = hipSuccess;
    uint32_t split = b.count;  // the longest come last
    while (split > 0 && b.tab.t[split - 1].logM / 2 >= 10) --split;
    // Rows of up to 2^9 alone, or rows of 2^10 alone: receive_pairs from four tiles of 2^13 points a compute unit on, or one of 2^14.  Whole calls (sender
    // too) in us, receive_tile / receive_pairs:
    // 2^13 points 256 73.6 / 74.3, 512 119 / 119.5, 768 164.6 / 166.6;  2^14 192 114 / 117.5, 256 142.7 / 145.1, 320 166.8 / 164.7,
    // 384 197.9 / 194.5, 512 197.3 / 193.1.  Both kinds are one launch of receive_pairs, which has one tail: a launch for either / one, ResNet-50 382 / 374,
    // random sets of 60 262 / 257, 100 451 / 438, 150 431 / 422 and 394 / 383, 200 741 / 732, 50 of 200 k and six of 2^21 266 / 255, 30 of 1 M and ten 471 / 462;
    // every XCD with its share of either kind (stretches.h), 30 of 70 k and 16 of 2^21 364 / 356, 24 513 / 483, 32 750 / 734, one of 2^16 and 24 485 / 457.
    auto pass = [&](auto kern, auto pairs, uint32_t pairs_from, unsigned lanes, size_t lds, size_t pairs_lds, uint32_t from, uint32_t end, int log_points) {
        const uint32_t total = long_starts(b, from, end, &at, [&](int logM) { return 1u << (logM - log_points); });
        const bool long_one = total >= pairs_from;
        if (long_one) {
            kern = pairs;
            lds = pairs_lds;
        }
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (err != hipSuccess) return err;
        const uint32_t few = from < split && split < end ? few_apart(total, at.at[split - from]) : 0u;
        FFTSP_LAUNCH("irfft_pass_b", kern, dim3(stretch_places(total, few)), dim3(long_one ? lanes : 1024u), lds, s, stream + 64, a.bits, a.m, entries, mid, t,
                     total, few, b.tab, at);
        return hipGetLastError();
    };
    const bool narrow = a.bits <= 8;
    if (e == hipSuccess && split > 0 && split < b.count)
        return pass(narrow ? k_receive_b_long<10, 16> : k_receive_b_long<10, 30>, narrow ? k_receive_pairs_long<10, 16> : k_receive_pairs_long<10, 30>, 0u,
                    HalfTile<10>::NT, Receive<10>::kLds, HalfTile<10>::kLds, 0, b.count, 14);
    if (e == hipSuccess && split > 0)
        e = pass(narrow ? k_receive_b_long<9, 16> : k_receive_b_long<9, 30>, narrow ? k_receive_pairs_long<9, 16> : k_receive_pairs_long<9, 30>, 1025u,
                 HalfTile<9>::NT, Receive<9>::kLds, HalfTile<9>::kLds, 0, split, 13);
    if (e == hipSuccess && split < b.count)
        e = pass(narrow ? k_receive_b_long<10, 16> : k_receive_b_long<10, 30>, narrow ? k_receive_pairs_long<10, 16> : k_receive_pairs_long<10, 30>, 257u,
                 HalfTile<10>::NT, Receive<10>::kLds, HalfTile<10>::kLds, split, b.count, 14);
    return e;
}

}  // namespace fftsp

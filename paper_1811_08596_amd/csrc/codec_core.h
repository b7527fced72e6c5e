// Device-side building blocks of selection, Algorithm 1 and packing (shared by the per-tile kernels in codec.hip and
// the chunk-resident kernels in chunk.hip).  Internal: nothing here is part of the C ABI.
#pragma once
#include "internal.h"
#include "record_bounds.h"

namespace fftsp {
namespace {

// The sign bit is masked: a finite sum of squares has none, and a NaN that carries one must still land inside the
// 31-bit key space the histogram and the radix digits are sized for (selection among non-finite bins is then
// ordinary integer work on their bit patterns, and exactly k bins survive whatever the input holds).
__device__ __forceinline__ uint32_t key_of(float2 z)
{
    return __float_as_uint(__fmaf_rn(z.x, z.x, __fmul_rn(z.y, z.y))) & 0x7FFFFFFFu;
}
__device__ __forceinline__ uint32_t vbits_of(float2 z)
{
    const uint32_t a = __float_as_uint(z.x) & 0x7FFFFFFFu, b = __float_as_uint(z.y) & 0x7FFFFFFFu;
    return a > b ? a : b;
}
// What is ranked and coded is either a complex frequency bin (two codes) or, for time-domain Top-k, a sample of
// the gradient itself (one code; the rank key is the bit pattern of |x|, an exact magnitude order).
__device__ __forceinline__ uint32_t key_of(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }
__device__ __forceinline__ uint32_t vbits_of(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }
template <bool REAL>
struct Elem {
    using T = float2;
    static constexpr uint32_t kCodes = 2;
    static __device__ __forceinline__ T zero() { return make_float2(0.f, 0.f); }
};
template <>
struct Elem<true> {
    using T = float;
    static constexpr uint32_t kCodes = 1;
    static __device__ __forceinline__ T zero() { return 0.f; }
};
// samples of chunk c that exist (time domain: the last chunk may end early, the rest counts as zeros)
template <bool REAL>
__device__ __forceinline__ uint32_t present_of(size_t n, size_t c, uint32_t B)
{
    if constexpr (REAL) {
        const size_t left = n - c * (size_t)B;
        return left < (size_t)B ? (uint32_t)left : B;
    } else {
        return B;
    }
}

// a plain 16-byte value that the compiler keeps in registers
typedef uint32_t u32x4 __attribute__((vector_size(16)));

// number of set bits of a wave-uniform mask below this lane (v_mbcnt_lo/hi: two instructions, no 64-bit math)
__device__ __forceinline__ uint32_t prefix_popc(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// What a kernel's input or output array holds: samples (time domain), or complex bins as binary32 or binary16 pairs.
template <bool REAL, bool HALF>
struct Stored {
    using T = typename Cx<HALF>::One;
};
template <bool HALF>
struct Stored<true, HALF> {
    using T = float;
};

// Scans and reductions over the 64 lanes with data-parallel-primitive moves (shifts within rows of 16 lanes, then
// broadcasts across rows): one instruction per step where a shuffle through LDS takes an address and a round trip.
// Lanes a move does not reach contribute zero.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t x)
{
    x += dpp_or_zero<0x111, 0xF>(x);  // row_shr:1
    x += dpp_or_zero<0x112, 0xF>(x);
    x += dpp_or_zero<0x114, 0xF>(x);
    x += dpp_or_zero<0x118, 0xF>(x);
    x += dpp_or_zero<0x142, 0xA>(x);  // lane 15 of rows 0 and 2 into rows 1 and 3
    x += dpp_or_zero<0x143, 0xC>(x);  // lane 31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_incl(v), 63);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    auto most = [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return a > b ? a : b; };
    v = most(v, dpp_or_zero<0x111, 0xF>(v));
    v = most(v, dpp_or_zero<0x112, 0xF>(v));
    v = most(v, dpp_or_zero<0x114, 0xF>(v));
    v = most(v, dpp_or_zero<0x118, 0xF>(v));
    v = most(v, dpp_or_zero<0x142, 0xA>(v));
    v = most(v, dpp_or_zero<0x143, 0xC>(v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// 32bit_to_Nbit of Algorithm 1 (value > max clamps to the top code; below eps flushes to the zero code)
__device__ __forceinline__ uint32_t quantize(uint32_t fbits, uint32_t pbase, int bits, int shift)
{
    if (bits == 32) return fbits;
    const int top = (1 << (bits - 1)) - 1;
    const int q = (int)((fbits & 0x7FFFFFFFu) >> shift) - (int)(pbase - 1u);  // both are below 2^31
    const int c = q < 0 ? 0 : (q > top ? top : q);
    const uint32_t sign = c ? (fbits >> 31) : 0u;
    return (sign << (bits - 1)) | (uint32_t)c;
}
// Nbit_to_32bit of Algorithm 1; bits of `code` above the lowest `bits` are ignored
__device__ __forceinline__ uint32_t dequantize(uint32_t code, uint32_t pbase, int bits, int shift)
{
    if (bits == 32) return code;
    const uint32_t c = code & ((1u << (bits - 1)) - 1u);
    const uint32_t v = ((c + (pbase - 1u)) << shift) | ((code << (32 - bits)) & 0x80000000u);
    return c ? v : 0u;
}

// The same for the code at bit `at` of a word, up to 16 bits wide; base = (pbase - 1) << shift.
__device__ __forceinline__ uint32_t dequantize_field(uint32_t word, uint32_t at, uint32_t bits, uint32_t base, int shift)
{
    const uint32_t c = __builtin_amdgcn_ubfe(word, at, bits - 1u);
    const uint32_t v = (((c << shift) + base) & 0x7FFFFFFFu) | ((word << (32u - bits - at)) & 0x80000000u);
    return c ? v : 0u;
}

// The tensor of a LongTable that this workgroup belongs to and its number in that tensor's share: one load by all lanes
// (a binary search would be six dependent ones).
struct LongShare {
    uint32_t tensor, blk;
};
__device__ __forceinline__ LongShare share_of(const uint16_t* at, uint32_t count, uint32_t workgroup)
{
    const uint32_t lane = threadIdx.x & 63u, start = lane < count ? (uint32_t)at[lane] : ~0u;
    const int i = (int)__popcll(__ballot(start <= workgroup)) - 1;
    return LongShare{(uint32_t)i, workgroup - (uint32_t)__builtin_amdgcn_readlane((int)start, i)};
}
__device__ __forceinline__ LongShare long_share(const LongStarts& at, uint32_t workgroup)
{
    LongShare share = share_of(at.at, at.count, workgroup);
    share.tensor += at.first;
    return share;
}
__device__ __forceinline__ LongShare long_share(const LongStarts& at) { return long_share(at, blockIdx.x); }

constexpr uint32_t kListCap = 256;  // keys of the threshold's bucket that are finished from a list

// The `need`-th largest of `count` listed keys that share all bits above `low`: tau grows bit by bit, a ballot counts
// the keys at or above each trial.  On return need = how many keys equal to tau are still to take, of `equal`.
// A trial that leaves exactly `need` keys ends the search: those are the ones.
template <int NR>
__device__ __forceinline__ void search_list(const uint32_t* list, uint32_t count, int low, int lane, uint32_t& tau,
                                            uint32_t& need, uint32_t& equal)
{
    uint32_t key[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) key[i] = (uint32_t)(lane + 64 * i) < count ? list[lane + 64 * i] : 0u;
    if (count == need) {
        equal = need;
        return;
    }
    for (int bit = low - 1; bit >= 0; --bit) {
        const uint32_t t = tau | (1u << bit);
        uint32_t cnt = 0;
#pragma unroll
        for (int i = 0; i < NR; ++i) cnt += (uint32_t)__popcll(__ballot(key[i] >= t));
        if (cnt >= need) tau = t;
        if (cnt == need) {
            equal = need;
            return;
        }
    }
    uint32_t above = 0;
    equal = 0;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        above += (uint32_t)__popcll(__ballot(key[i] > tau));
        equal += (uint32_t)__popcll(__ballot((uint32_t)(lane + 64 * i) < count && key[i] == tau));
    }
    need -= above;
}

// The two 32-bit codes of a kept bin.  They lie behind 16 bytes of header and W bitmap words, and W is odd for most chunk
// lengths, so words are all the alignment there is.
__device__ __forceinline__ uint2 load_code_pair(const uint32_t* p)
{
    uint2 v;
    __builtin_memcpy(&v, p, sizeof(v));
    return v;
}
__device__ __forceinline__ void store_code_pair(uint32_t* p, uint32_t re, uint32_t im)
{
    const uint2 v = make_uint2(re, im);
    __builtin_memcpy(p, &v, sizeof(v));
}

struct HeaderInfo {
    int write;
    uint64_t n;
    uint32_t L, C, N, m, k, S;
    float theta;
    uint32_t domain;  // 0: records hold frequency bins, 1: samples (time-domain Top-k)
    uint32_t scale;   // log2 of the factor on the spectrum (two's complement; half-precision variant), else 0
};
constexpr uint32_t kMagic = 0x31505346u;  // "FSP1"
// word i of the 64-byte stream header
__device__ __forceinline__ uint32_t header_word(const HeaderInfo& hdr, int i)
{
    switch (i) {
        case 0: return kMagic;
        case 1: return 1u;
        case 2: return (uint32_t)hdr.n;
        case 3: return (uint32_t)(hdr.n >> 32);
        case 4: return hdr.L;
        case 5: return hdr.C;
        case 6: return hdr.N;
        case 7: return hdr.m;
        case 8: return hdr.k;
        case 9: return hdr.S;
        case 10: return __float_as_uint(hdr.theta);
        case 11: return hdr.domain;
        case 12: return hdr.scale;
        default: return 0u;
    }
}
// whether a received stream header disagrees with what the caller asked for (theta is informative only)
__device__ __forceinline__ bool header_bad(const HeaderInfo& hdr, const uint32_t* __restrict__ h)
{
    bool bad = false;
    for (int i = 0; i < 13; ++i)
        if (i != 10) bad = bad || h[i] != header_word(hdr, i);
    return bad;
}

// 0, or 6 if a record (or the stream's header) is not what the call's arguments make it; kept: set bits of its bitmap
__device__ __forceinline__ uint32_t record_verdict(const uint8_t* __restrict__ record, const uint8_t* __restrict__ stream,
                                                   bool first_of_stream, uint32_t kept, uint32_t k, uint32_t word3,
                                                   const HeaderInfo& hdr)
{
    const uint32_t* rec = reinterpret_cast<const uint32_t*>(record);
    bool bad = kept != k || rec[2] != k || rec[3] != word3;
    if (hdr.write && first_of_stream) bad = bad || header_bad(hdr, reinterpret_cast<const uint32_t*>(stream));
    return bad ? 6u : 0u;
}

// what the first kernel of a receiver's call leaves in the control block
__device__ __forceinline__ void clear_control(uint32_t* __restrict__ ctl, const StatusNote& note, int tid, int lanes)
{
    // cleared as a whole: also the hand-over words of the fused inverse transform that may follow
    for (int i = tid; i < (int)(kControlBytes / 4); i += lanes)
        ctl[i] = i >= kNoteWord && i < kNoteWord + kNoteWords ? note_word(note, i) : 0u;
}

// A word every lane reads: by a scalar load, from memory that this kernel does not write.
template <typename T>
__device__ __forceinline__ T scalar_load(const T* p)
{
    return *(const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

// BINS neighbouring bins of one record: which of them are kept, and the stretch of the record their codes are in.
// WIDEST: bits of a bin at most (16: codes of up to 8, 30: of up to 15).
template <int BINS, int WIDEST>
struct Stretch {
    static constexpr int WORDS = (BINS * WIDEST + 31 + 31) / 32;
    uint32_t mask, rel;  // rel: bit position of the first code inside the window
    uint32_t w[WORDS];
    __device__ __forceinline__ void fetch(const uint32_t* codes, int final, uint32_t bit)
    {
        const int first = window_first(bit, final, WORDS);
        rel = bit - 32u * (uint32_t)first;
        __builtin_memcpy(w, codes + first, sizeof(w));
    }
    // put(j, word) for all bins: the code's two fields and what is above them, zero where one is not kept
    template <typename Put>
    __device__ __forceinline__ void unpack_codes(uint32_t twoN, Put&& put)
    {
        while (__any(rel >= 32u)) {  // windows moved back from a record's end
            const bool on = rel >= 32u;
#pragma unroll
            for (int i = 0; i + 1 < WORDS; ++i) w[i] = on ? w[i + 1] : w[i];
            w[WORDS - 1] = on ? 0u : w[WORDS - 1];
            rel = on ? (rel < 32u * WORDS ? rel - 32u : 0u) : rel;
        }
#pragma unroll
        for (int i = 0; i + 1 < WORDS; ++i) w[i] = __builtin_amdgcn_alignbit(w[i + 1], w[i], rel);
#pragma unroll
        for (int j = 0; j < BINS; ++j) {
            const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)mask, j, 1), raw = w[0] & m, by = m & twoN;
#pragma unroll
            for (int i = 0; i + 1 < WORDS; ++i)
                if (32 * i < (BINS - 1 - j) * WIDEST) w[i] = i + 2 < WORDS ? __builtin_amdgcn_alignbit(w[i + 1], w[i], by) : w[i] >> by;
            put(j, raw);
        }
    }
    // put(j, value) for all bins, zero where one is not kept
    template <typename Put>
    __device__ __forceinline__ void unpack(uint32_t twoN, uint32_t bits, int shift, uint32_t base, Put&& put)
    {
        asm("" : "+v"(base));  // in a vector register, so that it is the addend of a shift-and-add
        unpack_codes(twoN, [&](int j, uint32_t raw) __attribute__((always_inline)) {
            put(j, make_float2(__uint_as_float(dequantize_field(raw, 0u, bits, base, shift)),
                               __uint_as_float(dequantize_field(raw, bits, bits, base, shift))));
        });
    }
};

}  // namespace
}  // namespace fftsp

// The table of a record's bitmap that receivers read their bins by (receive.hip), for every kernel that makes one.
#pragma once
#include "codec_core.h"

namespace fftsp {
namespace {

constexpr int kTableLanes = 1024, kTableWaves = kTableLanes / 64;
__host__ __device__ constexpr uint32_t table_stride(int logM) { return (1u << (logM - 5)) + 2u; }  // entries, one to a bitmap word

// Entry i of a record's table: word i of its bitmap and the number of bits set before it.  A workgroup makes kTableWords of them
// and counts the words before its own itself, four loads in flight; the last one of a record leaves the record's verdict.
// (A workgroup per record: sixty records of 2^20 samples 10.8 -> 6.1 us, thirty-three of 2^22 39 -> 12.)
constexpr uint32_t kTableWords = 4 * kTableLanes;
__host__ __device__ constexpr uint32_t table_parts(int logM) { return ((1u << (logM - 5)) + kTableWords - 1u) / kTableWords; }
__device__ __forceinline__ void bitmap_part(const uint8_t* __restrict__ stream, const uint8_t* __restrict__ record, bool first_of_stream, uint32_t k,
                                            uint32_t word3, const HeaderInfo& hdr, int logM, uint32_t part, uint2* __restrict__ out,
                                            uint32_t* __restrict__ verdict)
{
    __shared__ uint32_t own[kTableWaves], earlier[kTableWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t parts = table_parts(logM);
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
    // every wave sums for itself, a lane to each of the others' sums
    const uint32_t one = lane < kTableWaves ? own[lane] : 0u, upto = wave_scan_incl(one), base = wave_sum(lane < kTableWaves ? earlier[lane] : 0u);
    const uint32_t all = base + (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    const uint32_t run = base + (uint32_t)__builtin_amdgcn_readlane((int)(upto - one), wave) + incl - sum;
    if (in) {
        const uint32_t r1 = run + (uint32_t)__popc(w.x), r2 = r1 + (uint32_t)__popc(w.y), r3 = r2 + (uint32_t)__popc(w.z);
        uint4* p = reinterpret_cast<uint4*>(out + 4u * at);  // the stride is even
        p[0] = make_uint4(w.x, run, w.y, r1);
        p[1] = make_uint4(w.z, r2, w.w, r3);
    }
    if (part + 1u == parts && tid == 0) {
        const uint32_t last = reinterpret_cast<const uint32_t*>(quads)[words];  // the Nyquist bin has a word to itself
        *reinterpret_cast<uint4*>(out + words) = make_uint4(last, all, 0u, 0u);
        *verdict = record_verdict(record, stream, first_of_stream, all + (uint32_t)__popc(last), k, word3, hdr);
    }
}
// where tensor i of a launch has its entries, in the spectrum's region
__device__ __forceinline__ size_t long_entries(const LongTensor& x, uint32_t i) { return (long_mid(x) >> 5) + 2u * i; }
// Part share.blk of tensor x, number share.tensor of its launch.
__device__ __forceinline__ void bitmap_part_of_tensor(const uint8_t* __restrict__ stream, const LongTensor& x, const LongShare& share, const HeaderInfo& hdr,
                                                      uint2* __restrict__ table, uint32_t* __restrict__ verdicts)
{
    bitmap_part(stream, stream + 64 + x.roff, share.tensor == 0, x.kept, 2u << x.logM, hdr, x.logM, share.blk, table + long_entries(x, share.tensor),
                verdicts + share.tensor);
}

}  // namespace
}  // namespace fftsp

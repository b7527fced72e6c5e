// Launchers of the chunk-resident codec (chunk.hip): chunk lengths up to 2^kChunkMaxLogL, one launch per direction.
#pragma once
#include "internal.h"

namespace fftsp {

constexpr int kChunkMaxLogL = 15;  // 2^14 complex values: 128 KiB of the 160 KiB a compute unit's LDS holds

// what select / pack / unpack need to know about a record
struct PackArgs {
    uint32_t k, W, S;      // kept units, bitmap words, record bytes
    uint32_t word3;        // 4th word of the record header
    uint32_t static_vmax;  // != 0: bit pattern of the caller's fixed range maximum
    int bits, m;
};

// Sender.  ctl: the workspace's control block.
hipError_t launch_chunk_compress(const float* in, size_t n, int logL, const CodecArgs& a, uint8_t* stream, uint8_t* records,
                                 uint32_t* ctl, Tables t, hipStream_t s);
// The same for time-domain Top-k.
hipError_t launch_topk_compress(const float* in, size_t n, int logL, const CodecArgs& a, uint8_t* stream, uint8_t* records,
                                uint32_t* ctl, hipStream_t s);
// Receiver.  streams: whole packed streams (64-byte header first).  plain: one stream, taken as it is; otherwise the
// streams are summed in list order, starting from zero.  verdicts: u32[npeers][C], announced by `note`.
hipError_t launch_chunk_decompress(const PeerList& streams, int npeers, int plain, int logL, const CodecArgs& a, float* out,
                                   size_t n, float gain, uint32_t* ctl, const StatusNote& note, uint32_t* verdicts, Tables t,
                                   hipStream_t s);

// Per-tensor calls: the tensors of up to 2^kChunkMaxLogL samples, longest first, cut into launches of kMaxTensors.  The
// table travels by value as a kernel argument (no host-to-device copy to order against the stream).
constexpr int kMaxTensors = 128;
struct TensorPiece {  // what one workgroup does: entries first .. first+count-1, all of 2^(logm+1) samples
    uint8_t first, count, logm, pad;
};
struct TensorTable {
    uint64_t goff[kMaxTensors];  // element offset of the tensor's first sample in the gradient
    uint64_t roff[kMaxTensors];  // byte offset of its record from the first record of the stream
    uint32_t glen[kMaxTensors];  // samples present; the rest of the chunk is zero
    TensorPiece piece[kMaxTensors];
    uint32_t kept[kChunkMaxLogL - 4], stride[kChunkMaxLogL - 4];  // kept bins and record bytes, by logm - 4
    uint32_t base;               // number of the table's first entry among all such tensors of the call
};
// From so many units of longer tensors on they have a stream of their own beside the shorter ones (api.hip, with the figures); below, their first kernel may be in
// the shorter ones' launch.
constexpr uint32_t kSideUnits = 1u << (23 - kLongUnitLog);
struct QuantizerArgs {
    int bits, m;
};
int tensors_per_workgroup(int logL);
// top_logL: the longest in the table; hdr: stream header (written or checked iff hdr.write_header).
// ctl (optional on the sender): the control block, cleared by the sender.
hipError_t launch_tensors_compress(const float* in, const TensorTable& t, uint32_t pieces, int top_logL, const QuantizerArgs& q,
                                   const CodecArgs& hdr, uint8_t* stream, uint8_t* records, uint32_t* ctl, Tables tb,
                                   hipStream_t s);
// note.count != 0: this launch leaves the note in the control block (clear: and clears the status word)
hipError_t launch_tensors_decompress(const uint8_t* stream, const TensorTable& t, uint32_t pieces, int top_logL,
                                     const QuantizerArgs& q, const CodecArgs& hdr, float* out, uint32_t* ctl,
                                     const StatusNote& note, int clear, uint32_t* verdicts, Tables tb, hipStream_t s);
// The same beside the first kernel of a few longer tensors, whose workgroups come behind theirs: one launch instead of two behind each other.
bool tensors_compress_beside(const TensorTable& t, const LongBatch& b);
bool tensors_decompress_beside(const TensorTable& t, uint32_t pieces, int bits, const LongBatch& b);
// and the forward pass A of b; clears zero_words at zero_ptr (launch_rfft_b_long goes on)
hipError_t launch_tensors_compress_beside(const float* in, const TensorTable& t, uint32_t pieces, const QuantizerArgs& q, const CodecArgs& hdr,
                                          uint8_t* stream, uint8_t* records, const LongBatch& b, float2* mid, uint32_t* zero_ptr, uint32_t zero_words,
                                          Tables tb, hipStream_t s);
// and, with verdicts of their own, b's inverse pass B out of the records, to mid (launch_inverse_a_long goes on), or, without short_decode, its records'
// table (launch_receive_b_long goes on)
hipError_t launch_tensors_decompress_beside(const uint8_t* stream, const TensorTable& t, uint32_t pieces, const QuantizerArgs& q, const CodecArgs& hdr,
                                            float* out, uint32_t* ctl, const StatusNote& note, uint32_t* verdicts, const LongBatch& b, float2* mid,
                                            void* table, uint32_t* long_verdicts, Tables tb, hipStream_t s);
// stage-level transforms, dense natural-order spectra
hipError_t launch_chunk_rfft(const float* in, size_t n, int logL, size_t C, float* spec, uint32_t sstride, Tables t,
                             hipStream_t s);
hipError_t launch_chunk_irfft(const float* spec, uint32_t sstride, size_t n, int logL, size_t C, float* out, Tables t,
                              hipStream_t s);

}  // namespace fftsp

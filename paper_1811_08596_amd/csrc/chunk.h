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

// A launch that decodes every record in one go has no earlier kernel that could clear the status word before a record
// raises it.  Such a launch stores one verdict per record instead, and this note in words 2..4 of the control block:
// how many there are, where (in words from the workspace's start), and a magic word.  fftsp_device_status looks at both.
struct StatusNote {
    uint32_t count, offset;
};
constexpr uint32_t kStatusNoteMagic = 0x46535653u;

// Sender.  a.tab != nullptr: per-tensor launch (records at a.tab->roff).  ctl (optional): the workspace's control block.
hipError_t launch_chunk_compress(const float* in, size_t n, int logL, const CodecArgs& a, uint8_t* stream, uint8_t* records,
                                 uint32_t* ctl, Tables t, hipStream_t s);
// Receiver.  streams: whole packed streams (64-byte header first).  plain: one stream, taken as it is; otherwise the
// streams are summed in list order, starting from zero.  verdicts (optional): u32[npeers][C], announced by `note`;
// nullptr: a bad record raises ctl[0], which is then not cleared here (a.write_header = check the stream header).
hipError_t launch_chunk_decompress(const PeerList& streams, int npeers, int plain, int logL, const CodecArgs& a, float* out,
                                   size_t n, float gain, uint32_t* ctl, const StatusNote& note, uint32_t* verdicts, Tables t,
                                   hipStream_t s);
// stage-level transforms, dense natural-order spectra
hipError_t launch_chunk_rfft(const float* in, size_t n, int logL, size_t C, float* spec, uint32_t sstride, Tables t,
                             hipStream_t s);
hipError_t launch_chunk_irfft(const float* spec, uint32_t sstride, size_t n, int logL, size_t C, float* out, Tables t,
                              hipStream_t s);

}  // namespace fftsp

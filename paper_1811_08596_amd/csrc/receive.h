// The receiver's decode and inverse pass B in one, long calls (receive.hip).
#pragma once
#include "internal.h"

namespace fftsp {

// whether a stream of C chunks of 2^(logM+1) samples can be received without a spectrum
bool receive_applies(int logM, size_t C, int bits);
// Fills mid.  stream: the 64-byte header and the records.  table: the spectrum's region of the workspace.  verdicts: u32[C], announced
// by note.
hipError_t launch_receive(const uint8_t* stream, const CodecArgs& a, int logM, void* table, float2* mid, Tables t, uint32_t* verdicts,
                          uint32_t* ctl, const StatusNote& note, hipStream_t s);

// The same for the tensors of a per-tensor launch (a.tab); first, if not null: the launch clears the control block and leaves it there.
bool receive_applies(const LongBatch& b, int bits);
hipError_t launch_receive_long(const uint8_t* stream, const CodecArgs& a, void* table, float2* mid, Tables t, int check_header, uint32_t* verdicts,
                               uint32_t* ctl, const StatusNote* first, hipStream_t s);

// its second kernel alone, where another launch has made the table (launch_tensors_decompress_beside)
hipError_t launch_receive_b_long(const uint8_t* stream, const CodecArgs& a, const void* table, float2* mid, Tables t, hipStream_t s);

}  // namespace fftsp

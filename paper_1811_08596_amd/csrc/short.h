// Launchers of the short calls' two-pass transforms (short.hip): chunk lengths 2^16 to 2^21.
#pragma once
#include "internal.h"

namespace fftsp {

// whether a call of C chunks of 2^(logM+1) samples, or a launch set of tensors, takes these kernels
bool short_forward(int logM, size_t C, int half);
bool short_forward(const LongBatch& b);
bool short_inverse(int logM, size_t C);
bool short_inverse(const LongBatch& b);

// as launch_rfft and its relatives (internal.h); mid_scale: what undoes or brings about the variant's lift (half_lift)
hipError_t launch_short_rfft(const float* in, size_t n, int logM, size_t C, float2* spec, uint32_t sstride, float2* mid, Tables t,
                             uint32_t* hist, uint32_t* zero_ptr, uint32_t zero_words, hipStream_t s);
hipError_t launch_short_rfft_half(const float* in, size_t n, int logM, size_t C, float2* spec, uint32_t sstride, float2* mid, Tables t,
                                  uint32_t* hist, uint32_t* zero_ptr, uint32_t zero_words, float in_scale, float mid_scale, hipStream_t s);
hipError_t launch_short_rfft_long(const float* in, const LongBatch& b, float2* spec, float2* mid, Tables t, uint32_t* hist,
                                  uint32_t* zero_ptr, uint32_t zero_words, hipStream_t s);
// its second pass alone
hipError_t launch_short_rfft_b_long(const LongBatch& b, float2* spec, const float2* mid, Tables t, uint32_t* hist, hipStream_t s);
// the inverse's two passes, B first
hipError_t launch_short_inverse_b(const float2* spec, uint32_t sstride, int logM, size_t C, float2* mid, Tables t, int pair_spec,
                                  hipStream_t s);
hipError_t launch_short_inverse_b_half(const float2* spec, uint32_t sstride, int logM, size_t C, float2* mid, Tables t, float mid_scale,
                                       hipStream_t s);
hipError_t launch_short_inverse_b_long(const float2* spec, const LongBatch& b, float2* mid, Tables t, hipStream_t s);
hipError_t launch_short_inverse_a(const float2* mid, int logM, size_t C, float* out, size_t n, Tables t, float gain, int half, hipStream_t s);
hipError_t launch_short_inverse_a_long(const LongBatch& b, float* out, const float2* mid, Tables t, hipStream_t s);

// The inverse pass B with the bins taken from the records: no launch that decodes, and no spectrum.
// verdicts, ctl, note: as launch_decode.
bool short_decode(int logM, size_t C);
bool short_decode(const LongBatch& b);
hipError_t launch_short_decode(const uint8_t* stream, const CodecArgs& a, int logM, float2* mid, Tables t, uint32_t* verdicts,
                               uint32_t* ctl, const StatusNote& note, hipStream_t s);
hipError_t launch_short_decode_long(const uint8_t* stream, const CodecArgs& a, float2* mid, Tables t, int check_header,
                                    uint32_t* verdicts, uint32_t* ctl, const StatusNote* first, hipStream_t s);

}  // namespace fftsp

// Where Top-k's threshold is looked for, from a sample of a chunk (codec.hip, k_sample).  Host code too, so that it can be checked there.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace fftsp {

constexpr uint32_t kSampleStretches = 2048, kSamples = 16u * kSampleStretches;
// where stretch g lies among the `slots` (a power of two) of its part
constexpr uint32_t sample_slot(uint32_t g, uint32_t slots) { return (g * 2654435761u >> 15) & (slots - 1u); }

// How much the sample's rank of the k-th largest of L varies, no less than that of samples drawn one by one.  differences: half the mean squared
// difference between neighbouring stretches' counts, times the stretches.  `present` of the L exist, and the zeros behind them, which are
// ranked too, are known: a chunk with few more than k samples in it has next to nothing left to vary.
constexpr float sample_variance(float differences, uint32_t k, uint32_t L, uint32_t present)
{
    const float left = k < present ? 1.f - (float)k / (float)present : 0.f, alone = (float)k / (float)L * left * (float)kSamples;
    return differences > alone ? differences : alone;
}

// and how far it can be off whatever the gradient is: a stretch at the gradient's end is in the sample or not
constexpr float sample_margin(uint32_t L, uint32_t present) { return present < L ? 20.f : 4.f; }

// Chunks of chunk_tiles tiles in a call of `tiles` of them; whole: the last one is full.
// Shorter chunks would have half or a quarter of their samples looked at, longer ones have more tiles than k_resolve holds the summaries of.
// Whole calls in us, histogram / sample, full chunks: 2^18 4224 tiles 50.4 / 51.8, 5888 59.6 / 61.4, 6656 66.8 / 67.3, 7680 75.0 / 73.4, 10240 89.9 / 84.6;  2^19 5888 63.6 /
// 65.1, 6656 69.7 / 70.4, 7680 78.5 / 76.9, 8960 86.1 / 83.8;  2^20 5120 65.8 / 67.1, 6144 72.3 / 74.0, 7168 81.0 / 80.9, 8192 87.2 / 87.3, 10240 100.0 / 96.3, 62 M samples 253 / 219.
// Where the last one is not, its zeros queue for one counter of the histogram, and are candidates where more is kept than there is: 2^20, nine chunks, the
// last 2, 5, 10, 16, 20, 30, 40, 50, 70, 90 % full, 126 / 66, 99 / 66, 98 / 66, 63 / 66, 71 / 69, 63 / 66, 69 / 64, 62 / 64, 73 / 64, 71 / 64; 2^18, forty, 73 / 58, 81 / 58, 77 /
// 58, 65 / 58, 56 / 59, 65 / 58, 60 / 57, 55 / 57, 57 / 57, 59 / 57.
constexpr bool sampled(uint32_t chunk_tiles, size_t tiles, bool whole) { return chunk_tiles >= 128 && chunk_tiles <= 513 && tiles > (whole ? 7168u : 4096u); }

}  // namespace fftsp

// Where Top-k's threshold is looked for, from a sample of a chunk (codec.hip, k_sample).  Host code too, so that it can be checked there.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace fftsp {

constexpr uint32_t kSamples = 1u << 15;
// The sample is stretches of so many neighbours, each out of an equal part of the chunk.  Neighbours are alike: shorter stretches know more, and longer ones
// are read faster.  Senders in us, histogram / stretches of sixteen / of eight, 15 and 50 % kept:
//   2^18 20 M samples, independent 67.4 / 53.0 / 55.2 and 72.4 / 58.0 / 60.8, rows of 1024 with a scale each 69.5 / 53.6 / 56.0 and 75.1 / 60.9 / 63.9, of 64 67.0 / 62.2 / 57.1 and 72.0 /
//     75.5 / 69.1, autoregressive (0.9) 68.7 / 55.1 / 56.7 and 72.5 / 59.8 / 61.6;
//   2^19 20 M 72.1 / 56.3 / 58.1 and 78.3 / 63.5 / 65.1, 73.1 / 57.5 / 59.9 and 77.1 / 66.1 / 68.1, 72.4 / 69.5 / 63.8 and 80.5 / 84.6 / 75.1, 75.2 / 61.5 / 62.3 and 78.1 / 67.8 / 67.1;
//   2^20 30 M 94.8 / 78.9 / 82.8 and 105.5 / 90.7 / 94.1, 96.5 / 94.3 / 83.3 and 103.9 / 119.5 / 99.1, 96.1 / 94.9 / 85.9 and 105.3 / 130.4 / 110.9, 93.9 / 80.8 / 84.2 and 105.7 / 93.9 / 96.1;
//     62 M 168.2 / 131.0 / 134.3 and 209.4 / 152.5 / 155.5, 166.3 / 143.7 / 134.1 and 207.2 / 180.0 / 160.7, 166.1 / 151.9 / 143.6 and 209.2 / 193.6 / 171.4; half of a sine 223 / 226 / 191.
// Of four, 62 M 144 where those of eight took 135.
constexpr uint32_t sample_stretch(uint32_t L) { return L >= 1u << 20 ? 8u : 16u; }
constexpr float kSampleDeviations = 4.5f;  // of the threshold's rank that are looked at, either side
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
constexpr float sample_margin(uint32_t L, uint32_t present) { return present < L ? 4.f + (float)sample_stretch(L) : 4.f; }

// Chunks of chunk_tiles tiles in a call of `tiles` of them; whole: the last one is full.
// Shorter chunks would have half or a quarter of their samples looked at, longer ones have more tiles than k_resolve holds the summaries of.
// Whole calls in us, 15 % kept at 32 bits, histogram / sample.  Full chunks: 2^18 5888 tiles 59.6 / 61.4, 6656 66.8 / 66.8, 7680 75.0 / 73.2, 10240 89.9 / 84.0;  2^19 5888 63.6 / 64.6,
// 6656 69.7 / 70.3, 7680 78.5 / 76.8, 10240 92.9 / 88.9;  2^20 8192 87.3 / 90.8, 10240 97.9 / 98.9, 15360 136.5 / 129.3, 20480 172.9 / 155.0.
// Where the last one is not, its zeros queue for one counter of the histogram, and are candidates where more is kept than there is: 2^20, nine chunks, the
// last 2, 5, 10, 16, 20, 30, 40, 50, 70, 90 % full, 125 / 66, 98 / 65, 99 / 66, 62 / 65, 71 / 68, 62 / 65, 70 / 65, 62 / 65, 73 / 66, 71 / 66; 2^19, twenty, 86 / 60, 85 / 60, 78 /
// 61, 60 / 60, 62 / 63, 66 / 59, 70 / 59, 59 / 59, 62 / 59, 70 / 60; 2^18, forty, 74 / 57, 80 / 57, 77 / 58, 62 / 57, 56 / 59, 66 / 57, 61 / 56, 55 / 56, 57 / 56, 59 / 56.
// Neighbours that are alike make the window wider, gradients on a grid crowd it, and the shortest of these calls lose.  Senders, rows of 64 with a scale each: 2^18 8.6 M 49.5 /
// 44.8, 2^19 9.1 M 47.5 / 54.7, 20.2 M 72.1 / 69.5, 2^20 8.9 M 50.0 / 67.1, 12.4 M 64.0 / 60.7, 30.3 M 94.0 / 85.4; rows of 1024: 2^20 8.9 M 51.3 / 55.1, 12.4 M 67.7 / 57.1; 8-bit
// floats: 2^18 8.6 M 95.2 / 81.5, 2^20 12.4 M 170.3 / 177.7, 40.3 M 246.6 / 233.8.
constexpr bool sampled(uint32_t chunk_tiles, size_t tiles, bool whole)
{
    return chunk_tiles >= 128 && chunk_tiles <= 513 && tiles > (!whole ? 4096u : chunk_tiles < 512 ? 7168u : 10240u);
}

}  // namespace fftsp

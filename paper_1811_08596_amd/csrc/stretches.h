// Which of a launch's tiles a workgroup does.  Workgroups are dealt out to the eight XCDs round-robin, and every XCD has a stretch of the tiles of
// its own, so that neighbours, which share lines, are in one L2.  Host code too, so that it can be checked there.
#pragma once
#include <stdint.h>

namespace fftsp {

constexpr uint32_t stretch_start(uint32_t xcd, uint32_t tiles) { return (uint32_t)((uint64_t)tiles * xcd >> 3); }
// tile of workgroup `place` of 8 * ceil(total / 8); at or above `total`: none
constexpr uint32_t stretch_tile(uint32_t place, uint32_t total)
{
    const uint32_t xcd = place & 7u, t = stretch_start(xcd, total) + (place >> 3);
    return t < stretch_start(xcd + 1u, total) ? t : total;
}
// The same where the first `few` tiles are of another kind, which take longer or less long: an XCD has its stretch of either.  With one stretch over both,
// one XCD has all of those few.  Sender and receiver in us of tensors whose rows are of 2^10 and shorter, the shorter ones first, one stretch / one of
// either: 30 of 70 k and 16 of 2^21 376 / 356, 24 511 / 483, 32 772 / 734 (a launch for either kind 751);  30 of 150 k and 24 541 / 513;  24 of 300 k and 24 566 / 552, 16 416 / 416.
// The shorter ones last: 24 and 32 488 and 734.
constexpr uint32_t stretch_tile(uint32_t place, uint32_t total, uint32_t few)
{
    const uint32_t xcd = place & 7u, i = place >> 3, mine = stretch_start(xcd + 1u, few) - stretch_start(xcd, few);
    if (i < mine) return stretch_start(xcd, few) + i;
    const uint32_t t = stretch_start(xcd, total - few) + i - mine;
    return t < stretch_start(xcd + 1u, total - few) ? few + t : total;
}
// One kind, with the XCDs beginning their stretches `step` tiles further into a tensor each, and going round (0: where they start).  For passes whose tiles are a few
// columns of a tensor, 128 tiles to the longest: their rows are 8 KiB apart, and XCDs that are at the same columns of tensors a power of two apart ask the same channels of the
// memory.  Forward pass A of tensors' senders, sender in us, each from its stretch's start / this (in brackets a persistent kernel that dealt the tiles out
// otherwise): 2^21 16 208.3 / 199.8 (201.7), 24 276 / 277 (289), 28 317 / 316 (333), 32 363 / 352 (355), 48 572 / 552 (558);  2^22 four 132 / 127 (134), eight 227 / 209 (225),
// sixteen 374 / 372 (394).  An eighth of the stretch further each: 28 of 2^21 324, 12 and thirty of 70 k 183 where this takes 177.
constexpr uint32_t kTurnStep = 16;
constexpr uint32_t turned_tile(uint32_t place, uint32_t total, uint32_t step)
{
    const uint32_t xcd = place & 7u, lo = stretch_start(xcd, total), hi = stretch_start(xcd + 1u, total), t = lo + (place >> 3);
    if (t >= hi) return total;
    const uint32_t to = t + (step ? ((step * xcd - lo) & (8u * step - 1u)) % (hi - lo) : 0u);
    return to < hi ? to : to - (hi - lo);
}
// How many of a launch's first `few` tiles have stretches of their own: up to three tenths of the launch.  More lie on several XCDs anyhow, and the order of the passes before and
// after is worth more.  Sender and receiver in us of random sets of tensors, one stretch / one of either, by share: 23 % 692 / 684, 24 % 376 / 366, 27 % 269 / 266, 29 % 336 / 334;
// 31 % 468 / 476, 35 % 389 / 395, 36 % 445 / 463, 45 % 451 / 459 and 432 / 440.
constexpr uint32_t few_apart(uint32_t total, uint32_t few) { return 10u * few < 3u * total ? few : 0u; }
// workgroups that have a tile for everyone
constexpr uint32_t stretch_places(uint32_t total, uint32_t few = 0) { return 8u * ((few + 7u) / 8u + (total - few + 7u) / 8u); }

}  // namespace fftsp

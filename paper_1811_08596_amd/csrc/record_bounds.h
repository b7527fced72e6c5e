// Which of a record's words a receiver reads for a code, counted from its first code word (the bitmap lies before it).  A corrupt
// bitmap's ranks point anywhere; these stay inside the record.  Host code too, so that it can be checked there.
#pragma once
#include <stdint.h>

namespace fftsp {

// of a record of S bytes with W bitmap words; -1: there is none
constexpr int last_code_word(uint32_t S, uint32_t W) { return (int)(S / 4u) - 5 - (int)W; }
// The word that bit `bit` of the codes is in, and the one after it.  last: not below zero.
constexpr int code_word(uint32_t bit, int last) { return (int)(bit >> 5) < last ? (int)(bit >> 5) : last; }
constexpr int word_after(int word, int last) { return word < last ? word + 1 : word; }
// First of `words` words, that word among them unless it lies outside the record; below zero: in the bitmap.
constexpr int window_first(uint32_t bit, int last, int words) { return code_word(bit, last - (words - 1)); }

}  // namespace fftsp

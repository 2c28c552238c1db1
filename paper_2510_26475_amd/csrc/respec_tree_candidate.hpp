// Which bytes the tree sampler reads for the two logits of a candidate.  Plain C++, so that the rule can be tested on the
// host.
#pragma once

#include <cstdint>

namespace respec {

// A logit may come with the rest of its aligned 32-bit word (the scalar cache has no narrower load) where that
// word is part of the row: always in fp32, and in rows that are whole, aligned 16-byte slots.  In any other row of 16-bit
// logits the word can reach two bytes beyond it, and so beyond the caller's buffer: those are read by themselves.
constexpr bool candidate_by_word(bool bf16, bool whole_rows) { return !bf16 || whole_rows; }

constexpr uint64_t candidate_word_at(uint64_t row, int x, bool bf16) { return (row + (uint64_t)x * (bf16 ? 2 : 4)) & ~(uint64_t)3; }

// The bits of a logit (as binary32) in its word.
constexpr uint32_t candidate_bits(uint32_t word, uint64_t row, int x, bool bf16) {
    return !bf16 ? word : (row + (uint64_t)x * 2) & 2 ? word & 0xffff0000u : word << 16;
}

}  // namespace respec

"""Which bytes the tree sampler reads for a candidate's logit (host-side: the rule is plain C++, compiled here with g++).

For rows at every alignment that the entry point takes and every candidate, the read has to stay inside the row and
give that logit's bits.
"""
import os
import shutil
import subprocess

import pytest

from paper_2510_26475_amd import build

PROGRAM = r"""
#include "respec_tree_candidate.hpp"
#include <cstdio>
#include <cstring>

int main() {
    alignas(16) static unsigned char memory[256];
    for (int i = 0; i < 256; ++i) memory[i] = (unsigned char)(17 * i + 3);
    long reads = 0, by_word = 0, outside = 0, wrong = 0;
    for (int bf16 = 0; bf16 < 2; ++bf16)
        for (int V = 1; V <= 40; ++V)
            for (int at = 16; at < 32; at += bf16 ? 2 : 4) {
                const int size = bf16 ? 2 : 4;
                const uint64_t row = (uint64_t)(memory + at), end = row + (uint64_t)V * size;
                const bool whole = at == 16 && V * size % 16 == 0;
                for (int x = 0; x < V; ++x) {
                    uint32_t want = 0;
                    std::memcpy((char *)&want + (4 - size), memory + at + x * size, size);
                    ++reads;
                    if (!respec::candidate_by_word(bf16, whole)) continue;  // read by itself
                    ++by_word;
                    const uint64_t word_at = respec::candidate_word_at(row, x, bf16);
                    if (word_at < row || word_at + 4 > end) {
                        ++outside;
                        continue;
                    }
                    uint32_t word;
                    std::memcpy(&word, (const void *)word_at, 4);
                    if (respec::candidate_bits(word, row, x, bf16) != want) ++wrong;
                }
            }
    std::printf("%ld %ld %ld %ld\n", reads, by_word, outside, wrong);
}
"""


def test_a_candidates_logit_is_read_inside_its_row(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    src = tmp_path / "candidate.cpp"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, str(src), "-o", str(tmp_path / "candidate")], check=True)
    out = subprocess.run([str(tmp_path / "candidate")], capture_output=True, text=True, check=True).stdout
    reads, by_word, outside, wrong = (int(x) for x in out.split())
    assert outside == 0 and wrong == 0
    assert reads == 820 * (4 + 8) and by_word == 820 * 4 + 8 + 16 + 24 + 32 + 40  # fp32, and bf16 in whole rows


def test_the_library_is_built_again_when_the_rule_changes():
    assert os.path.join(build.CSRC, "respec_tree_candidate.hpp") in build._inputs()

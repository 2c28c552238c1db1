"""Which members of a distillation team are waited for (host-side: the bookkeeping is plain C++, compiled here with g++).

One member's view of a team of eight over 64 rows: the others answer a few ticks after they are asked, member 3 not at all
for some of the rows.  The wait for it has to be paid in full once and not on every row, and it has to be waited for again
once it answers.
"""
import os
import shutil
import subprocess

import pytest

from paper_2510_26475_amd import build

PROGRAM = r"""
#include "respec_kd_absent.hpp"
#include <cstdio>

// ticks spent on a row; given: the members given up on it
static long row(respec::KdAbsent &a, const long (&answers_after)[8], long spin, unsigned &given) {
    given = 0;
    for (long t = 0;; ++t) {
        unsigned late = 0;
        for (int m = 1; m < 8; ++m)
            if (answers_after[m] > t && !(given >> m & 1)) late |= 1u << m;
        if (late == 0) {
            a.row_done();
            return t;
        }
        given |= a.give_up(late, (uint64_t)t, (uint64_t)spin);
    }
}

int main() {
    const long spin = 5000, never = 1L << 40;
    respec::KdAbsent a;
    for (int r = 0; r < 64; ++r) {
        long after[8];
        for (int m = 0; m < 8; ++m) after[m] = 10 + (m * 7 + r) % 50;
        if (r >= 8 && r < 40) after[3] = never;
        if (r == 50) after[5] = 400;   // slow, within the wait
        unsigned given;
        const long t = row(a, after, spin, given);
        std::printf("%d %ld %u\n", r, t, given);
    }
    respec::KdAbsent b;                // a wait of nothing: everybody is given up at the first look
    const long after[8] = {0, 5, 5, 5, 5, 5, 5, 5};
    unsigned given;
    const long t = row(b, after, 0, given);
    std::printf("64 %ld %u\n", t, given);
}
"""


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("kd_absent")
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", f"-I{build.CSRC}", str(d / "t.cpp"), "-o", str(d / "t")], check=True)
    out = subprocess.run([str(d / "t")], check=True, capture_output=True, text=True, timeout=60).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def test_a_member_that_does_not_run_costs_one_wait(rows):
    waits = [t for r, t, given in rows if 8 <= r < 40]
    assert waits[0] == 5001 and all(t == 5000 // 16 + 1 for t in waits[1:])  # (the look after the decision counts)
    assert all(given == 1 << 3 for r, _, given in rows if 8 <= r < 40)


def test_members_that_answer_are_waited_for(rows):
    for r, t, given in rows[:64]:
        if not 8 <= r < 40:
            assert given == 0, r       # the first row that member 3 answers on among them
            assert t == (400 if r == 50 else max(10 + (m * 7 + r) % 50 for m in range(1, 8))), r


def test_a_wait_of_nothing_gives_everybody_up(rows):
    assert rows[64] == (64, 1, 0xfe)


def test_the_library_is_built_again_when_the_bookkeeping_changes():
    assert os.path.join(build.CSRC, "respec_kd_absent.hpp") in build._inputs()

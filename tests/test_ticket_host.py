"""The ticket that tells a launch's last block (csrc/ticket.hpp), compiled for the host and its memory operations put in orders as mixed as can be."""
import subprocess

import pytest

from paper_2512_07710_amd.build import CSRC, HIPCC

PROGRAM = r"""
#include "ticket.hpp"
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
using namespace moe355;
struct Launches {                                              // the blocks that have yet to arrive; before any operation others may do theirs
    std::mt19937 rng{1};
    std::vector<int> waiting;                                  // blocks, by launch
    int word = 0, n = 0, lasts = 0;
    struct Count {
        Launches& l;
        void others() const { while (l.rng() % 4 != 0 && l.arrive()) {} }
        int increment(int limit) const {
            others();
            const int v = l.word;
            l.word = (unsigned)v >= (unsigned)limit ? 0 : v + 1;
            return v;
        }
        int add(int v) const { others(); l.word += v; return l.word - v; }
        void store(int v) const { others(); l.word = v; }
    };
    bool arrive() {
        if (waiting.empty()) return false;
        waiting.pop_back();
        lasts += ADD_AND_STORE ? with_a_store(Count{*this}) : last_to_arrive(Count{*this}, n);
        return true;
    }
    bool with_a_store(const Count& c) {
        if (c.add(1) != n - 1) return false;
        c.store(0);
        return true;
    }
    void run(int launches) {
        waiting.assign(launches * n, 0);
        lasts = 0;
        while (arrive()) {}
    }
};
int main() {
    int bad = 0, alone = 0;
    Launches l;
    for (l.n = 1; l.n <= 64; ++l.n)
        for (int i = 0; i < 200; ++i) {
            for (int launches = 1; launches <= 3; ++launches) {
                l.run(launches);
                (launches == 1 ? alone : bad) += l.word != 0 || l.lasts != launches;
                l.run(1);                                      // the call behind
                (launches == 1 ? alone : bad) += l.word != 0 || l.lasts != 1;
                l.word = 0;
            }
        }
    printf("%d %d\n", alone, bad);
    return 0;
}
"""


@pytest.mark.parametrize("add_and_store", [0, 1])
def test_a_launch_has_one_last_block_whatever_ran_before(add_and_store, tmp_path):
    """Launches of 1 to 64 blocks alone, and two or three that overlap, then one alone: one last block each, and the ticket at zero.  (The same
    search finds an add that the last block follows with a store of zero: sound alone, and off zero for good once launches overlap.)"""
    (tmp_path / "ticket.hip").write_text(PROGRAM)
    subprocess.run([HIPCC, "--cuda-host-only", "-O2", "-std=c++17", f"-DADD_AND_STORE={add_and_store}", "-I", CSRC, str(tmp_path / "ticket.hip"), "-o",
                    str(tmp_path / "ticket")], check=True, capture_output=True)
    alone, overlapped = map(int, subprocess.run([str(tmp_path / "ticket")], check=True, capture_output=True, text=True).stdout.split())
    assert alone == 0 and (overlapped > 0) == bool(add_and_store)

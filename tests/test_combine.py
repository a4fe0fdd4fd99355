"""The slot sequence of the gradient combining tables (csrc/combine.hpp), compiled for the host and run on the keys a
wave of 64 cells meets: consecutive dofs, and dofs that lie a stride apart."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include <cstdio>
#include <cstdlib>
#include "combine.hpp"
using namespace coffee::dev;
// args: slots, first key, stride, keys. Prints every key's slots in probe order, then the slots the keys take when
// they are inserted one after the other (-1: given up) and the number of probes in all.
int main(int, char** v) {
    const unsigned ts = atoi(v[1]);
    const unsigned long long k0 = atoll(v[2]), st = atoll(v[3]);
    const int n = atoi(v[4]);
    bool* taken = (bool*)calloc(ts, 1);
    long probes = 0;
    for (int i = 0; i < n; ++i) {
        unsigned s = combine_first(k0 + i * st, ts);
        int got = -1;
        for (int t = 0; t < kCombineProbes; ++t) {
            if (t) s = combine_next(s, ts);
            printf("%u ", s);
            if (got < 0) {
                ++probes;
                if (!taken[s]) { taken[s] = true; got = (int)s; }
            }
        }
        printf("%d\\n", got);
    }
    printf("%ld\\n", probes);
    free(taken);
}
"""


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    d = tmp_path_factory.mktemp("combine")
    src, exe = d / "probe.cpp", d / "probe"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1407_0904_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)

    def run(slots, first, stride, n):
        out = subprocess.run([str(exe), str(slots), str(first), str(stride), str(n)], check=True, capture_output=True,
                             text=True).stdout.strip().split("\n")
        rows = [[int(x) for x in line.split()] for line in out[:-1]]
        return [r[:-1] for r in rows], [r[-1] for r in rows], int(out[-1])

    return run


@pytest.mark.parametrize("slots", [128, 256])
def test_probes_reach_different_slots(table, slots):
    """No probe of a key is spent on a slot that it has seen, and all slots are in the table."""
    for first in (0, 5, 1 << 20, (1 << 31) - 9):
        seqs, _, _ = table(slots, first, 1, 16)
        for s in seqs:
            assert len(set(s)) == len(s) and min(s) >= 0 and max(s) < slots


@pytest.mark.parametrize("stride", [1, 2, 8, 64, 1000])
@pytest.mark.parametrize("slots", [128, 256])
def test_half_full_table_takes_every_key(table, slots, stride):
    """Half as many keys as slots find a place, in a few probes each, whatever the stride of the dof numbers."""
    for first in (0, 3, 123456):
        _, got, probes = table(slots, first, stride, slots // 2)
        assert min(got) >= 0
        assert probes <= 3 * len(got), probes


@pytest.mark.parametrize("slots", [128, 256])
def test_consecutive_keys_are_neighbours(table, slots):
    """A group of eight consecutive keys lies in one aligned group of eight slots."""
    _, got, _ = table(slots, 8 * 1234, 1, 8)
    assert len({g // 8 for g in got}) == 1 and len(set(got)) == 8

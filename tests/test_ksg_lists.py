"""CPU check of the bounds of a KSG walk (csrc/ksg_lists.hpp): whatever an order and the
words that it leaves unwritten hold, a walk reads inside its pair's lists and ends at their
outermost sentinels at the latest; on prepared orders the bounds change nothing."""
import os
import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parents[1] / "paper_2307_02203_amd" / "csrc"
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "ksg_lists.hpp"
using namespace ndf;

static long reads_out = 0, endless = 0, changed = 0, walks = 0;

// Both sides of a walk over `lists` (walked codes) from block starts L and R, at the k-th
// distance that stops latest; a side whose block leaves the region counts and ends.
static void walk(const std::vector<int> &lists, int me, int L, int R) {
    const int n = (int)lists.size();
    ++walks;
    for (int side = 0; side < 2; ++side) {
        int at = side ? R : L, steps = 0;
        for (;;) {
            if (at < 0 || at + kPad > n) { ++reads_out; break; }
            if (++steps > n) { ++endless; break; }
            const unsigned d = side ? (unsigned)lists[at + kPad - 1] - (unsigned)me
                                    : (unsigned)me - (unsigned)lists[at];  // wraps as on the GPU
            if ((int)d >= kUnset) break;
            at += side ? kPad : -kPad;
        }
    }
}

int main(int argc, char **argv) {
    const int N = atoi(argv[1]);
    const int n0 = atoi(argv[2]), n1 = N - n0, E = list_entries(N);
    std::mt19937 rng(N + n0);
    // prepared orders: y ranks of the x order's samples
    std::vector<int> jr(N);
    for (int i = 0; i < N; ++i) jr[i] = i;
    std::shuffle(jr.begin(), jr.end(), rng);
    std::vector<int> seen(2 * E, 0);
    for (int order = 0; order < 2; ++order) {
        std::vector<int> other(N);
        for (int i = 0; i < N; ++i) other[order ? jr[i] : i] = order ? i : jr[i];
        int q1 = 0;
        for (int r = 0; r < N; ++r) {
            const bool up = other[r] >= n0;
            const int at = list_place(up, r, q1, n0, n1) + order * E;
            const int there = place_sum(order * E, n0, r) - at;
            if (walk_place(at, E) != at || walk_other(there, E) != there) ++changed;
            if ((int)start_place(pack_start(at, 12345)) != at) ++changed;
            if (start_gap(pack_start(at, kTopCode)) != kTopCode) ++changed;
            ++seen[kPad + at];
            q1 += up;
        }
        for (int pad = 0; pad < 4; ++pad)
            for (int u = 0; u < kPad; ++u) ++seen[pad_place(pad, order * E, n0, n1) + u];
    }
    for (int s : seen)
        if (s != 1) ++changed;  // entries and sentinels tile the region
    // anything between the sentinels, starts from any 16-bit word and any sum of entries
    const int fills[] = {0, 1, kTopCode, kFar, -kFar, 2147483647, -2147483647 - 1, -(1 << 30)};
    for (int fill = 0; fill < 10; ++fill) {
        std::vector<int> lists(2 * E);
        for (int &c : lists) c = fill < 8 ? fills[fill] : fill == 8 ? (int)rng() : (int)(rng() % kTopCode);
        for (int order = 0; order < 2; ++order)
            for (int pad = 0; pad < 4; ++pad)
                for (int u = 0; u < kPad; ++u)
                    lists[pad_place(pad, order * E, n0, n1) + u] = pad_code(pad);
        for (int word = 0; word < 65536; word += N > 300 ? 17 : 1) {
            const int at = kPad + walk_place(start_place(pack_start(word, (int)rng())), E);
            const int me = walk_code(lists[at]);
            walk(lists, me, at - kPad, at + 1);
            const int there = kPad + walk_other((int)(rng() % 200000) - 100000, E);
            walk(lists, me, there - kPad, there);
        }
    }
    for (int m = 0; m < 65536; ++m) {
        const int got = order_member((uint16_t)m, N);
        if (got < 0 || got >= N || (m < N && got != m)) ++changed;
    }
    printf("%ld %ld %ld %ld\n", walks, reads_out, endless, changed);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("ksg_lists")
    (d / "walk.hip").write_text(PROGRAM)
    exe = d / "walk"
    subprocess.run([HIPCC, "--offload-host-only", "-O2", "-std=c++17", f"-I{CSRC}",
                    str(d / "walk.hip"), "-o", str(exe)], check=True, capture_output=True)
    return exe


@pytest.mark.parametrize("n_members,n0", [(2, 1), (3, 1), (5, 2), (64, 32), (64, 63), (257, 128),
                                          (257, 1), (1000, 500), (1000, 930), (2048, 1024)])
def test_walks_stay_in_the_lists(program, n_members, n0):
    r = subprocess.run([str(program), str(n_members), str(n0)], capture_output=True, text=True, check=True,
                       timeout=100)
    walks, reads_out, endless, changed = map(int, r.stdout.split())
    assert walks > 10000
    assert reads_out == 0 and endless == 0
    assert changed == 0

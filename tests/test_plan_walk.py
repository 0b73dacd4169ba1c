"""The search that finds the end of a micro-batch (csrc/plan_walk.h), compiled for the host and run with a loop over the
lanes where the device counts a ballot: next-fit's own answer, and no place asked for beyond the shard's end."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_13833_amd", "csrc")
HARNESS = r"""
#include <algorithm>
#include <cstdint>
#define __device__
#define __forceinline__ inline
using std::max; using std::min;
#include "plan_walk.h"
// The starts of the micro-batches of n slots (pre[0 .. n]: tokens before a slot); -1 if a place outside 0 .. n is asked for.
extern "C" int walk(int lg_G, int n, const int64_t* pre, int64_t budget, int32_t* starts) {
    const int G = 1 << lg_G;
    int m = 0, j = 0, sz = 0;
    bool outside = false;
    while (j < n && !outside) {
        starts[m++] = j;
        const int64_t limit = pre[j] + budget;
        const int e = dc::next_fit_end(G, lg_G, j, sz, n, [&](int c0, int step, int last, bool inside) {
            int cnt = 0;
            for (int lane = 0; lane < G; ++lane) {
                const int c = c0 + lane * step;
                if (inside && c > last) continue;
                const int at = min(c, last);
                if (at < 0 || at > n) { outside = true; continue; }
                cnt += pre[at] <= limit ? 1 : 0;
            }
            return cnt;
        });
        sz = e - j;
        j = e;
    }
    return outside ? -1 : m;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan_walk")
    (d / "walk.cpp").write_text(HARNESS)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "walk.so"), str(d / "walk.cpp")])
    lib = C.CDLL(str(d / "walk.so"))

    def run(lens, budget, lg):
        pre = np.concatenate([[0], np.cumsum(lens, dtype=np.int64)])
        starts = np.zeros(len(lens) + 1, np.int32)
        m = lib.walk(lg, len(lens), pre.ctypes.data_as(C.c_void_p), C.c_int64(budget), starts.ctypes.data_as(C.c_void_p))
        return None if m < 0 else starts[:m].tolist()
    return run


def _next_fit(lens, budget):
    starts, load = [], budget + 1
    for j, ln in enumerate(lens):
        if load + ln > budget:
            starts.append(j)
            load = 0
        load += int(ln)
    return starts


@pytest.mark.parametrize("lg", [4, 5, 6])
def test_micro_batches_of_a_shard(walk, lg):
    rng = np.random.default_rng(lg)
    shapes = [np.concatenate([np.full(100, 10), np.full(50, 500)]),       # the rest is shorter than the micro-batch before it ...
              np.concatenate([np.full(4000, 1), np.full(70, 999)]),       # ... and does not fit
              np.full(1000, 7), np.arange(1, 700), np.arange(700, 0, -1), np.array([5]), np.full(64, 2000)]
    for _ in range(200):
        n = int(rng.integers(1, 600))
        lens = rng.integers(1, int(rng.choice([2, 20, 400])), n)
        shapes.append(np.sort(lens) if rng.random() < 0.4 else lens)
    for lens in shapes:
        for budget in (1, 30, 1000, 12345, 10**7):
            assert walk(lens, budget, lg) == _next_fit(lens, budget), (lens[:8], len(lens), budget)

"""CPU check of the eigensolver's ranking rule (csrc/rank.h, plain C++): the
places are a permutation in descending order, NaN and infinities included."""
import itertools
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_05900_amd", "csrc")

SOURCE = r"""
#include <cstdio>
#include <vector>
#include "rank.h"
int main() {
    int n;
    while (std::scanf("%d", &n) == 1) {
        std::vector<double> v(n);
        for (double& x : v) std::scanf("%lf", &x);
        for (int i = 0; i < n; ++i) {
            int parts = 0;   // eight lanes, as the kernels share the count
            for (int r = 0; r < 8; ++r) parts += hotrg::entries_before(v.data(), n, i, r, 8);
            std::printf("%d %d ", hotrg::descending_place(v.data(), n, i), parts);
        }
        std::printf("\n");
    }
}
"""


def places(tmp_path, rows):
    """Per row of values, the places and the same counted by eight lanes."""
    (tmp_path / "t.cpp").write_text(SOURCE)
    exe = tmp_path / "t"
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__host__=", "-D__device__=", "-I", CSRC, str(tmp_path / "t.cpp"),
                    "-o", str(exe)], check=True)
    text = "\n".join(f"{len(v)} " + " ".join(repr(x) for x in v) for v in rows)
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(out) == len(rows)
    return [np.array(line.split(), dtype=int).reshape(-1, 2) for line in out]


def test_places_are_a_permutation_whatever_the_values(tmp_path):
    rows = [list(v) for n in range(1, 6) for v in itertools.product([float("nan"), float("inf"), 5.0, 0.0, -float("inf")],
                                                                    repeat=n)]
    rng = np.random.default_rng(1)
    for n in (16, 81, 96):
        v = rng.integers(0, 9, n).astype(float)
        v[rng.integers(0, n, n // 4)] = np.nan
        rows.append(v.tolist())
    for v, got in zip(rows, places(tmp_path, rows)):
        assert (got[:, 0] == got[:, 1]).all()
        key = np.where(np.isnan(v), -np.inf, v)
        want = np.empty(len(v), dtype=int)
        want[np.lexsort((np.arange(len(v)), -key))] = np.arange(len(v))
        assert (got[:, 0] == want).all(), v


def test_places_of_a_padded_block(tmp_path):
    """p values, some NaN, padded with minus infinity to 96: the first p take
    the places 0 .. p - 1 (the order in which a block's columns are kept)."""
    rng = np.random.default_rng(2)
    rows = []
    for p in (32, 48, 80, 96):
        for share in (0.0, 0.3, 1.0):
            v = np.where(rng.random(p) < share, np.nan, rng.standard_normal(p))
            rows.append(v.tolist() + [-float("inf")] * (96 - p))
    for v, got in zip(rows, places(tmp_path, rows)):
        p = 96 - v.count(-float("inf"))
        assert sorted(got[:p, 0]) == list(range(p))

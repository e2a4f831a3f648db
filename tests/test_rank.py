"""CPU checks of the eigensolver's ranking rules (csrc/rank.h, plain C++): the
places are a permutation in descending order, and the largest entry's row is
one of the column's, NaN and infinities included."""
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
        for (double& x : v) {
            std::scanf("%lf", &x);
            x = hotrg::rankable(x);   // as the kernels store what they rank
        }
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


LARGEST = r"""
#include <cstdio>
#include <vector>
#include "rank.h"
int main() {
    int n, stride;
    while (std::scanf("%d %d", &n, &stride) == 2) {
        std::vector<double> v((size_t)n * stride, 1e9);   // other columns: not to be read as this one's
        for (int i = 0; i < n; ++i) std::scanf("%lf", &v[(size_t)i * stride]);
        std::vector<hotrg::Entry> e;
        for (int t = 0; t < 256; ++t) e.push_back(hotrg::largest_entry(v.data(), stride, n, t, 256));
        for (int s = 128; s > 0; s >>= 1)
            for (int t = 0; t < s; ++t) e[t] = hotrg::larger_entry(e[t], e[t + s]);
        std::printf("%d\n", e[0].row);
    }
}
"""


def test_largest_entry_is_a_row_of_the_column(tmp_path):
    (tmp_path / "t.cpp").write_text(LARGEST)
    exe = tmp_path / "t"
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__host__=", "-D__device__=", "-I", CSRC, str(tmp_path / "t.cpp"),
                    "-o", str(exe)], check=True)
    rng = np.random.default_rng(3)
    rows = [[float("nan")] * n for n in (1, 4, 255, 256, 257, 2304)]
    for n in (1, 2, 81, 256, 300, 2304):
        for share in (0.0, 0.5):
            v = rng.integers(-5, 6, n).astype(float)      # ties: the lowest row
            rows.append(np.where(rng.random(n) < share, np.nan, v).tolist())
    text = "\n".join(f"{len(v)} 3 " + " ".join(repr(x) for x in v) for v in rows)
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.split()
    for v, got in zip(rows, map(int, out), strict=True):
        size = np.where(np.isnan(v), -1.0, np.abs(v))
        assert 0 <= got < len(v)
        if not np.isnan(v).all():
            assert got == int(np.argmax(size))

"""CPU check of the Jacobi rounds' stopping rule (csrc/jacobi_rule.h, plain
C++): the rounds emulated in 80-bit arithmetic, with the header's tests, end
with every pair's cosine at most the rotation tolerance and the drift that
the header states."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_05900_amd", "csrc")

# P columns with norms 10^(-spread j / P) and pairwise cosines +-c: odd-even
# rounds (a pair changes places after its rotation) until P in a row make no
# large rotation, as jacobi_rounds does
SOURCE = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "jacobi_rule.h"
typedef long double real;
int main(int argc, char** argv) {
    const int P = atoi(argv[1]);
    const real spread = strtold(argv[2], 0), c0 = strtold(argv[3], 0);
    const int signs = atoi(argv[4]);
    const double tol = atof(argv[5]), tol2 = tol * tol;
    std::vector<std::vector<real>> a(P, std::vector<real>(P, 0));
    unsigned seed = 7;
    for (int p = 0; p < P; ++p)
        for (int q = p; q < P; ++q) {
            seed = seed * 1664525u + 1013904223u;
            const real s = signs && (seed >> 31) ? -1 : 1;
            a[p][q] = a[q][p] = p == q ? 1 : s * c0 / 2;
        }
    for (int p = 0; p < P; ++p)
        for (real& x : a[p]) x *= powl(10.0L, -spread * p / P);
    auto dot = [&](int p, int q) {
        real s = 0;
        for (int i = 0; i < P; ++i) s += a[p][i] * a[q][i];
        return s;
    };
    int rd = 0, last = -1;
    for (; rd - 1 - last < P && rd < 40 * P; ++rd)
        for (int p = rd & 1; p + 1 < P; p += 2) {
            const int q = p + 1;   // y at p, x at q
            const real nx = dot(q, q), ny = dot(p, p), ga = dot(p, q);
            real c = 1, s = 0;
            if (hotrg::jacobi_rotates((double)(ga * ga), (double)(nx * ny), tol2)) {
                const real d = ny - nx, y = 1 / sqrtl(d * d + 4 * ga * ga);
                c = sqrtl(0.5L * fabsl(d) * y + 0.5L);
                s = (d >= 0 ? ga : -ga) * y / c;
                if (hotrg::jacobi_large((double)(ga * ga), (double)(nx * ny), (double)(s * s))) last = rd;
            }
            for (int i = 0; i < P; ++i) {
                const real x = a[q][i], v = a[p][i];
                a[p][i] = c * x - s * v;
                a[q][i] = s * x + c * v;
            }
        }
    real worst = 0;
    for (int p = 0; p < P; ++p)
        for (int q = p + 1; q < P; ++q) worst = fmaxl(worst, fabsl(dot(p, q)) / sqrtl(dot(p, p) * dot(q, q)));
    printf("%d %.6Le %.6e\n", rd, worst, hotrg::jacobi_drift(P));
}
"""


@pytest.fixture(scope="module")
def rounds(tmp_path_factory):
    d = tmp_path_factory.mktemp("jacobi")
    (d / "t.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__host__=", "-D__device__=", "-I", CSRC, str(d / "t.cpp"), "-o",
                    str(d / "t")], check=True)

    def run(*args):
        out = subprocess.run([str(d / "t"), *map(str, args)], capture_output=True, text=True, check=True).stdout.split()
        return int(out[0]), float(out[1]), float(out[2])
    return run


# the eigensolver's tolerance at its widths, the chain update's at its widest;
# cosines on both sides of the line between small and large rotations
@pytest.mark.parametrize("P,tol", [(32, 4e-15), (64, 4e-15), (96, 4e-15), (64, 1e-14)])
@pytest.mark.parametrize("spread", [6, 12])
@pytest.mark.parametrize("cosine", [1.1e-8, 9e-9, 1.9e-9, 3e-15])
@pytest.mark.parametrize("signs", [0, 1])
def test_rounds_end_within_the_stated_bound(rounds, P, tol, spread, cosine, signs):
    n, worst, drift = rounds(P, spread, cosine, signs, tol)
    assert n < 40 * P
    assert worst <= tol + drift


def test_the_tolerance_alone_is_not_the_bound(rounds):
    """One sweep of small rotations can leave more than the tolerance."""
    n, worst, _ = rounds(96, 12, 9e-9, 0, 4e-15)
    assert n == 96 and worst > 4e-15

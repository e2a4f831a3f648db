// When the one-sided Jacobi rounds (jacobi.h) rotate a pair and when they end.
// Plain C++: the rule is the same on the host.
#pragma once

namespace hotrg {

// A rotation is large if the pair's cosine is above 1e-8 or the rotation's sine
// above 3.2e-8.  The rounds end after a sweep without a large rotation; a
// further one would only confirm that next to nothing rotates any more (it
// took Ritz matrices at p = 48 from 80 to 92 us, dense n = 64 from 241 to 258, 32
// updates of 512 chains of chi = 30 from 11.2 to 12.0 ms).
constexpr double JAC_LARGE_COS2 = 1e-16, JAC_LARGE_SIN2 = 1e-15;

// What the rounds leave: a pair's cosine is at most the rotation tolerance when
// the pair meets, and until the sweep ends either of its columns turns with
// each of the others at most once.  A small rotation of columns x, y moves the
// cosine of x with a third column z by at most max(sine, |y| / |x| sine) times
// the cosine of y, z, where |y| / |x| times the sine is at most 1.5 times the
// sine or twice the cosine of x, y.  So every cosine is at most the tolerance
// plus this: 9e-14 for 96 columns, 6e-14 for 64 (8e-15 is the most that
// matrices made for it, with all cosines at 9e-9, were seen to end with).
constexpr double jacobi_drift(int columns) { return 2.0 * (columns - 2) * (1.5 * 3.17e-8 * 1e-8); }

// ga2: squared dot product, nn: product of the squared norms, s2: squared sine
__host__ __device__ inline bool jacobi_rotates(double ga2, double nn, double tol2) { return ga2 > tol2 * nn; }
__host__ __device__ inline bool jacobi_large(double ga2, double nn, double s2) {
    return ga2 > JAC_LARGE_COS2 * nn || s2 > JAC_LARGE_SIN2;
}

}  // namespace hotrg

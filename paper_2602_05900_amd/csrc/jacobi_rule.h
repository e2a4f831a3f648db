// When the one-sided Jacobi rounds (jacobi.h) rotate a pair and when they end.
// Plain C++: the rule is the same on the host.
#pragma once

namespace hotrg {

// A rotation is large if the pair's cosine or the rotation's sine is above
// JAC_LARGE.  The rounds end after a sweep without a large rotation: a further
// one, which would only confirm that nothing rotates any more, is not needed,
// because a pair's cosine is at most the rotation tolerance when the pair meets
// and drifts little afterwards.  A small rotation of columns x, y moves the
// cosine of x with a third column z by at most
//   max(sine, |y| / |x| sine) cosine(y, z) <= 2 JAC_LARGE^2
// (|y| / |x| times the sine is the cosine of x, y, for |y| >> |x|, and at most
// twice it or 1.5 times the sine in between), and until the sweep ends either
// column of a pair turns with each of the others at most once.
constexpr double JAC_LARGE = 2e-9;
constexpr double jacobi_drift(int columns) { return 2.0 * (columns - 2) * (2.0 * JAC_LARGE * JAC_LARGE); }

// Squared rotation tolerance that leaves every pair of `columns` columns with a
// cosine of at most tol.
constexpr double jacobi_tol2(double tol, int columns) {
    return (tol - jacobi_drift(columns)) * (tol - jacobi_drift(columns));
}

// ga2: squared dot product, nn: product of the squared norms, s2: squared sine
__host__ __device__ inline bool jacobi_rotates(double ga2, double nn, double tol2) { return ga2 > tol2 * nn; }
__host__ __device__ inline bool jacobi_large(double ga2, double nn, double s2) {
    return ga2 > (JAC_LARGE * JAC_LARGE) * nn || s2 > JAC_LARGE * JAC_LARGE;
}

}  // namespace hotrg

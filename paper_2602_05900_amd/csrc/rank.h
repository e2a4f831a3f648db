// Places in descending order, for the eigensolver's kernels.  Plain C++: the
// rule is the same on the host.
#pragma once

namespace hotrg {

// How many of v[first], v[first + step], ... (below n) stand before entry i in
// descending order, ties by index; with first = 0 and step = 1, entry i's
// place.  A NaN counts as minus infinity, so the places are a permutation of
// 0 .. n - 1 whatever the values: they are used as row and column numbers,
// also in a solve that ends as failed because its values are not finite.
__host__ __device__ inline int entries_before(const double* v, int n, int i, int first, int step) {
    const double lowest = -__builtin_inf();
    const double mine = v[i] == v[i] ? v[i] : lowest;
    int count = 0;
    for (int j = first; j < n; j += step) {
        const double other = v[j] == v[j] ? v[j] : lowest;
        count += other > mine || (other == mine && j < i) ? 1 : 0;
    }
    return count;
}

__host__ __device__ inline int descending_place(const double* v, int n, int i) {
    return entries_before(v, n, i, 0, 1);
}

}  // namespace hotrg

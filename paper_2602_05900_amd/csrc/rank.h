// Places in descending order and the largest entry of a column, for the
// eigensolver's and the chain update's kernels.  Plain C++: the rules are the
// same on the host.
#pragma once

namespace hotrg {

// A value as it is ranked: a NaN counts as minus infinity, so that the places
// below are a permutation of 0 .. n - 1 whatever the values.  They are used as
// row and column numbers, also in a solve that ends as failed because its
// values are not finite.
__host__ __device__ inline double rankable(double v) { return v == v ? v : -__builtin_inf(); }

// How many of v[first], v[first + step], ... (below n, rankable) stand before
// entry i in descending order, ties by index; with first = 0 and step = 1,
// entry i's place.
__host__ __device__ inline int entries_before(const double* v, int n, int i, int first, int step) {
    const double mine = v[i];
    int count = 0;
    for (int j = first; j < n; j += step) count += (v[j] > mine) || (v[j] == mine && j < i) ? 1 : 0;
    return count;
}

__host__ __device__ inline int descending_place(const double* v, int n, int i) {
    return entries_before(v, n, i, 0, 1);
}

// An entry of a column by magnitude and row.
struct Entry {
    double size;
    int row;
};

// a unless b is larger, or as large and in a lower row
__host__ __device__ inline Entry larger_entry(const Entry& a, const Entry& b) {
    return b.size > a.size || (b.size == a.size && b.row < a.row) ? b : a;
}

// The largest of v[i stride], i = first, first + step, ... below n (n > 0).
// Where none compares (all NaN, or no such i) its row is still one of the
// column's, since the entry found is read again for its sign.
__host__ __device__ inline Entry largest_entry(const double* v, long stride, int n, int first, int step) {
    Entry e{-1.0, first < n ? first : n - 1};
    for (int i = first; i < n; i += step) {
        const double a = __builtin_fabs(v[(long)i * stride]);
        if (a > e.size) e = Entry{a, i};
    }
    return e;
}

}  // namespace hotrg

// FP64 top-k eigensolver of the symmetric environment E (n x n) on the device.
//
// The truncation of a HOTRG step keeps the leading k eigenvectors of
// E = M M^T, to which the higher-order SVD of the merged tensor reduces
// (Sec. II.A).  Only k << n of them are needed, so for n > P_MAX the solver
// is a block subspace iteration, alternating power and Ritz passes on an
// n x p block (p > k):
//
//   power:  Z = E X;  G = Z^T Z = D^-1 L L^T D^-1 (columns scaled to unit
//           norm by D);  V <- Z D L^-T  (CholeskyQR)
//   Ritz:   W = E V;  G = W^T W = D^-1 L L^T D^-1, so W = Q R with
//           R^T = D^-1 L;  R^T J = S diag(sigma) by one-sided Jacobi:
//           S holds the right singular vectors of W = E V, and
//           u = V S are the Ritz vectors, W S = E u, sigma = |E u|;
//           residual |E u_j - sigma_j u_j|;  V <- u;  converged? else the
//           next power pass starts from X = E u / sigma
//
// (sigma_j u_j against E u_j: to first order the same residual as with the
// Rayleigh quotient.)  Both passes need one Gram matrix, which the product
// kernel leaves in partial sums, and its Cholesky factor; the Ritz pass
// costs the Jacobi besides.  R^T is graded with nearly orthogonal columns
// once V is near the eigenvectors, so the Jacobi takes 3-4 sweeps there.
// Warm-started from the Ritz block of the step two earlier (same fused leg
// basis once the dims are steady), else from a counter-based random block.
// For n <= P_MAX the environment is diagonalised completely.
//
// The rotations are the paper's plane rotations of index pairs (Sec. II.B,
// Eqs. (5)-(6), Fig. 3), each pair meeting once a sweep in a systolic
// exchange, applied from one side to a factor of the matrix.
//
// All reductions are in a fixed order (no atomics), so a solve is bitwise
// reproducible.
#include <math.h>
#include "common.h"
#include "jacobi.h"
#include "rank.h"
#include "../../include/hotrg.h"

namespace hotrg {

constexpr int EIG_PMAX = kEigPMax; // largest Ritz block / fully diagonalised matrix
constexpr int EIG_ROWS = kEigRows; // rows of the block one workgroup handles
constexpr int EIG_MAX_SWEEPS = 40;
// A Ritz pass (and the convergence test) every second pass: the span of the
// block, on which convergence depends, grows the same way in either, and a
// Ritz pass costs the Jacobi more (every third pass misses the bound in 30
// passes).
constexpr int EIG_RR_EVERY = 2;
// Scaled Gram matrices whose Cholesky pivots stay above EIG_PIV_OK are
// factored as they are; else (nearly dependent columns: the first pass from
// a random block, or kept pairs in the rounding noise) with EIG_SHIFT on the
// diagonal, which bounds |L^-1| by 3e6.
constexpr double EIG_PIV_OK = 1e-11, EIG_SHIFT = 1e-13;
// Ritz vectors below this fraction of the largest sigma enter the next power
// pass as u, not as E u / sigma: the product's rounding (1e-16 of the
// largest) leaves in E u / sigma a part 1e-16 / f along the leading vectors
// (f = sigma over the largest), which the next product raises to 1e-16 / f^2
// of the column itself: nothing at f = 1e-7, but a nearly dependent column
// below 1e-8, whose factor then tilts the leading vectors (at 1e-10 the deep
// ordered phase, T = 1.8 and D = 48, ended at residuals of 3e-8 after 100
// passes; now below 1e-12 after 68).
constexpr double EIG_ADVANCE = 1e-7;
constexpr double EIG_MU = 1e-15;   // shift of a warm-started solve, relative to Tr E

// ---------------------------------------------------------------- helpers

__device__ __forceinline__ bool eig_done(const EigCtl* c) { return c->done != 0; }

// splitmix64 hash of a counter -> uniform double in [-1, 1)
__device__ __forceinline__ double hash_uniform(unsigned long long x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    x = x ^ (x >> 31);
    return (double)(x >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// ---------------------------------------------------------------- init

// Trace of E, control reset; fills V with random columns unless warm.
__global__ __launch_bounds__(256) void eig_init_kernel(const double* __restrict__ E, int n, double* __restrict__ V,
                                                       int p, int warm, unsigned long long seed, EigCtl* ctl) {
    __shared__ double sh[256];
    if (blockIdx.x == 0) {
        double t = 0.0;
        for (int i = threadIdx.x; i < n; i += 256) t += E[(long)i * n + i];
        sh[threadIdx.x] = t;
        __syncthreads();
        for (int s = 128; s > 0; s >>= 1) {
            if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            ctl->trace = sh[0];
            ctl->done = 0;
            ctl->iters = 0;
            ctl->converged = 0;
            ctl->resid = 0.0;
            ctl->best = 1e300;
            ctl->stall = 0;
            ctl->jac_capped = 0;
        }
    }
    if (!warm) {
        const long total = (long)n * p;
        const double unit = sqrt(3.0 / n);   // columns of norm about 1
        for (long e = blockIdx.x * 256L + threadIdx.x; e < total; e += (long)gridDim.x * 256)
            V[e] = unit * hash_uniform(seed * 0x100000001B3ull + (unsigned long long)e);
    }
}

// ---------------------------------------------------------------- Y = E X and its Gram matrix

// doubles of one workgroup's partial Gram matrix: the 16 x 16 tiles (i, j),
// i <= j, of the p x p matrix, in that order
__host__ __device__ constexpr int gram_tiles(int nf) { return nf * (nf + 1) / 2; }
__device__ __forceinline__ int gram_tile(int nf, int i, int j) { return i * nf - i * (i - 1) / 2 + (j - i); }

// Gram tiles of 16 staged rows by NW waves, into the workgroup's slot of part.
template <int NF, int NW>
__device__ __forceinline__ void gram_rows(const double (*xs)[16 * NF + 2], double* __restrict__ part) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, fr = lane & 15, fk = lane >> 4;
    double* out = part + (long)blockIdx.x * (gram_tiles(NF) * 256);
    int t = 0;
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
        for (int j = i; j < NF; ++j, ++t) {
            if (t % NW != wave) continue;
            d4 g = d4{0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                g = __builtin_amdgcn_mfma_f64_16x16x4f64(xs[fk + 4 * q][16 * i + fr], xs[fk + 4 * q][16 * j + fr], g, 0,
                                                         0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) out[t * 256 + (fk + 4 * q) * 16 + fr] = g[q];
        }
}

// Workgroup: EIG_ROWS = 16 rows of Y = (E + mu I) X (n x p, p = 16 NF), all columns;
// the 8 waves split K, reduce through LDS, and the workgroup's part of
// Y^T Y follows from the rows while they are there (no pass over Y for it).
// A lane takes 4 consecutive k of its row per 16 (E read as 32 contiguous
// bytes a lane, whole lines a wave), the next 16 loaded while the current
// ones are multiplied.  Bound by those loads' latency at small n and by the
// reads of E and X at large n: 8.2 / 18 / 40 us at n = 576 / 1024 / 2304,
// p = 48 / 64 / 80, Gram part included (15.6 / 28 / 68 us, and 9 / 13 / 19 us
// for a pass over Y, with four waves, no loads ahead and separate kernels).
template <int NF>
__global__ __launch_bounds__(512) void eig_ev_kernel(const double* __restrict__ E, int n,
                                                     const double* __restrict__ X, double* __restrict__ Y,
                                                     double* __restrict__ part, double mu_rel, const EigCtl* ctl) {
    if (eig_done(ctl)) return;
    constexpr int P = 16 * NF, LD = P + 2, NW = 8;
    const double mu = mu_rel * ctl->trace;
    typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
    __shared__ double red[NW][EIG_ROWS][LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r0 = blockIdx.x * EIG_ROWS;
    const int fr = lane & 15, fk = lane >> 4;
    d4 acc[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = d4{0, 0, 0, 0};
    const int chunk = ((n + 16 * NW - 1) / (16 * NW)) * 16;
    const int kb = wave * chunk, ke = min(n, kb + chunk);
    const double* erow = E + (long)min(r0 + fr, n - 1) * n;
    auto load = [&](int k, double (&a)[4], double (&b)[4][NF]) {
        const int k0 = k + 4 * fk;
        const d2u e0 = *reinterpret_cast<const d2u*>(erow + k0), e1 = *reinterpret_cast<const d2u*>(erow + k0 + 2);
        a[0] = e0.x;
        a[1] = e0.y;
        a[2] = e1.x;
        a[3] = e1.y;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int f = 0; f < NF; ++f) b[u][f] = X[(long)(k0 + u) * P + f * 16 + fr];
    };
    auto multiply = [&](const double (&a)[4], const double (&b)[4][NF]) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[f] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u][f], acc[f], 0, 0, 0);
    };
    const int full = ke > kb ? (ke - kb) / 16 : 0;   // whole groups of 16
    if (full > 0) {
        double a[4], b[4][NF];
        load(kb, a, b);
        for (int i = 1; i < full; ++i) {
            double a2[4], b2[4][NF];
            load(kb + 16 * i, a2, b2);
            multiply(a, b);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a[u] = a2[u];
#pragma unroll
                for (int f = 0; f < NF; ++f) b[u][f] = b2[u][f];
            }
        }
        multiply(a, b);
    }
    const int kt = kb + 16 * full;
    if (kt < ke) {   // the last, partial group (n not a multiple of 16)
        double a[4], b[4][NF];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = kt + 4 * fk + u;
            const bool in = k < ke;
            a[u] = in ? erow[k] : 0.0;
#pragma unroll
            for (int f = 0; f < NF; ++f) b[u][f] = in ? X[(long)k * P + f * 16 + fr] : 0.0;
        }
        multiply(a, b);
    }
    // component q of lane l holds row (l/16) + 4q, column l%16 of each tile
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int q = 0; q < 4; ++q) red[wave][fk + 4 * q][f * 16 + fr] = acc[f][q];
    __syncthreads();
    for (int e = tid; e < EIG_ROWS * P; e += 512) {
        const int r = e / P, c = e - (e / P) * P;
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += red[w][r][c];
        if (r0 + r < n) {
            v = fma(mu, X[(long)(r0 + r) * P + c], v);
            Y[(long)(r0 + r) * P + c] = v;
        } else {
            v = 0.0;   // rows past n add nothing to the Gram matrix
        }
        red[0][r][c] = v;   // read by this thread only, above
    }
    __syncthreads();
    gram_rows<NF, NW>(red[0], part);
}

// The workgroup's part of X^T X alone.
template <int NF>
__global__ __launch_bounds__(64 * NF) void eig_gram_kernel(const double* __restrict__ X, int n,
                                                           double* __restrict__ part, const EigCtl* ctl) {
    if (eig_done(ctl)) return;
    constexpr int P = 16 * NF;
    __shared__ double xs[EIG_ROWS][P + 2];
    const long r0 = (long)blockIdx.x * EIG_ROWS;
    for (int e = threadIdx.x; e < EIG_ROWS * P; e += 64 * NF) {
        const int r = e / P, c = e - (e / P) * P;
        xs[r][c] = r0 + r < n ? X[(r0 + r) * P + c] : 0.0;
    }
    __syncthreads();
    gram_rows<NF, NF>(xs, part);
}

// out[e] = sum_b part[b][e] for e < count (a multiple of 32): 32 elements a
// workgroup, eight threads each, in a fixed order.
__global__ __launch_bounds__(256) void eig_sum_kernel(const double* __restrict__ part, int nb, int count,
                                                      double* __restrict__ out, const EigCtl* ctl) {
    if (eig_done(ctl)) return;
    __shared__ double sh[8][32];
    const int c = threadIdx.x & 31, seg = threadIdx.x >> 5;
    const int e = blockIdx.x * 32 + c;
    double s = 0.0;
#pragma unroll 4
    for (int b = seg; b < nb; b += 8) s += part[(long)b * count + e];
    sh[seg][c] = s;
    __syncthreads();
    if (seg == 0) {
#pragma unroll
        for (int i = 1; i < 8; ++i) s += sh[i][c];
        out[e] = s;
    }
}

// ---------------------------------------------------------------- small Cholesky

// Blocked Cholesky factorisation A = L L^T of a symmetric P x P matrix in LDS
// (P = 16 NF, row stride P + 1; the lower triangle is used), by NF waves.
// A 16-column panel is factored by wave 0 in registers (lane = row, the
// pivot row through readlane: no barrier and no LDS on the column chain),
// the trailing blocks are then updated by all waves on the matrix cores.
// Pivots below `floor` are raised to it.  linv receives 1 / L_jj, *minp the
// smallest pivot met.  Ends with a barrier.
template <int NF>
__device__ __forceinline__ void chol_blocked(double* A, double floor, double* linv, double* minp) {
    constexpr int P = 16 * NF, LDA = P + 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 15, fk = lane >> 4;
    if (tid == 0) *minp = 1e300;
    for (int b = 0; b < NF; ++b) {
        const int j0 = 16 * b;
        if (wave == 0) {
            const int row0 = j0 + lane, row1 = row0 + 64;
            const bool in0 = row0 < P, in1 = row1 < P;
            double x[16], y[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                x[c] = in0 ? A[row0 * LDA + j0 + c] : 0.0;
                y[c] = in1 ? A[row1 * LDA + j0 + c] : 0.0;
            }
            double mp = 1e300;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                double piv = readlane_d(x[j], j);
                mp = fmin(mp, piv);
                piv = fmax(piv, floor);
                const double rs = rsqrt_nr(piv);
                const double inv = rs * rs;
                const double mx = x[j] * inv, my = y[j] * inv;
#pragma unroll
                for (int c = j + 1; c < 16; ++c) {
                    const double v = readlane_d(x[j], c);
                    x[c] = fma(-mx, v, x[c]);
                    y[c] = fma(-my, v, y[c]);
                }
                x[j] = lane == j ? piv * rs : x[j] * rs;
                y[j] *= rs;
                if (lane == 0) linv[j0 + j] = rs;
            }
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                if (in0 && (lane >= 16 || c <= lane)) A[row0 * LDA + j0 + c] = x[c];
                if (in1) A[row1 * LDA + j0 + c] = y[c];
            }
            if (lane == 0) *minp = fmin(*minp, mp);
        }
        __syncthreads();
        // trailing blocks (i, j), b < j <= i, dealt to the waves in turn
        int t = 0;
        for (int i = b + 1; i < NF; ++i)
            for (int j = b + 1; j <= i; ++j, ++t) {
                if (t % NF != wave) continue;
                d4 acc;
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] = A[(16 * i + fk + 4 * q) * LDA + 16 * j + fr];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-A[(16 * i + fr) * LDA + j0 + fk + 4 * q],
                                                               A[(16 * j + fr) * LDA + j0 + fk + 4 * q], acc, 0, 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q) A[(16 * i + fk + 4 * q) * LDA + 16 * j + fr] = acc[q];
            }
        __syncthreads();
    }
}

// Mailboxes and keys of one workgroup's Jacobi rounds over P columns of P
// rows; the Cholesky matrix and the mailboxes are never live together.
template <int NF>
struct SmallEig {
    static constexpr int P = 16 * NF, G = P / 2, LDA = P + 1;
    static constexpr int SLOT = P + 8;   // 8 modulo 16 doubles: the groups of a wave spread over the banks
    static constexpr int DOUBLES = 2 * G * SLOT > P * LDA ? 2 * G * SLOT : P * LDA;
    double buf[DOUBLES];
    double nrm[2 * G];
    double key[P];
    double linv[P];
    double minp;
    int flag[2];
};

// rotate while |a_p.a_q| > 4e-15 |a_p| |a_q| (what the rounds leave: jacobi_rule.h)
constexpr double EIG_JAC_TOL2 = 1.6e-29;

// ---------------------------------------------------------------- dense eigenproblem

// E of an early step (n <= EIG_PMAX) diagonalised completely, one workgroup:
// the rows and columns sorted by descending diagonal, the Cholesky factor of
// E + mu I (mu = 1e-15 Tr E; a thousand times larger while a pivot says that
// E, whose products may be in a split precision, is not definite to that
// accuracy), and one-sided Jacobi on the factor's columns: their norms are
// sqrt(lambda + mu), their directions the eigenvectors, orthogonal whatever
// the rank of E.  theta[j] descending, S column j the matching eigenvector
// (row-major n x n).
//
// Bound by the rounds' dependent chain (jacobi.h).  The factor's columns are
// graded and nearly orthogonal, so 6-7 sweeps do (the two-sided method took
// 10 on E itself), on one matrix instead of two, with one barrier a round
// instead of two: n = 64 took 876 us two-sided, 250 to 280 us now (259 in a
// solve with D = 8; where the loop comes to lie in memory moves it by 10 %).
template <int NF>
__global__ __launch_bounds__(64 * NF) void eig_dense_kernel(const double* __restrict__ E, int n,
                                                            double* __restrict__ theta, double* __restrict__ S,
                                                            EigCtl* ctl) {
    using Sh = SmallEig<NF>;
    constexpr int P = Sh::P, LDA = Sh::LDA, RL = 2 * NF;
    __shared__ Sh sh;
    __shared__ int place[P];    // place[i]: row of E at sorted position i
    const int tid = threadIdx.x, g = tid >> 3, r = tid & 7;
    // sorted order of the diagonal, descending, ties by index
    for (int i = tid; i < P; i += 64 * NF) sh.key[i] = i < n ? rankable(E[(long)i * n + i]) : 0.0;
    __syncthreads();
    double trace = 0.0;
    for (int i = 0; i < n; ++i) trace += sh.key[i];
    for (int i = tid; i < n; i += 64 * NF) place[descending_place(sh.key, n, i)] = i;
    __syncthreads();
    double mu = 1e-15 * fabs(trace);
    for (int attempt = 0;; ++attempt) {
        for (int e = tid; e < P * P; e += 64 * NF) {
            const int i = e / P, j = e - (e / P) * P;
            double v = i == j ? 1.0 : 0.0;
            if (i < n && j < n) {
                const long a = place[i], b = place[j];
                v = 0.5 * (E[a * n + b] + E[b * n + a]) + (i == j ? mu : 0.0);
            }
            sh.buf[i * LDA + j] = v;
        }
        __syncthreads();
        chol_blocked<NF>(sh.buf, fmax(1e-3 * mu, 1e-280), sh.linv, &sh.minp);
        const bool good = sh.minp >= 0.25 * mu;
        __syncthreads();
        if (good || attempt == 5) break;
        mu *= 1e3;
    }
    double x[RL], y[RL];
#pragma unroll
    for (int i = 0; i < RL; ++i) {
        const int row = r + 8 * i, c = 2 * g;
        y[i] = row < n && c < n && c <= row ? sh.buf[row * LDA + c] : 0.0;
        x[i] = row < n && c + 1 < n && c + 1 <= row ? sh.buf[row * LDA + c + 1] : 0.0;
    }
    if (tid < 2) sh.flag[tid] = -1;
    __syncthreads();
    bool capped;
    unsigned nrot = 0;
    const int G = (n + 1) / 2;
    const JacobiShared js{sh.buf, sh.nrm, sh.flag, Sh::SLOT};
    const int rounds = jacobi_rounds<RL, false>(x, y, js, G, g, r, EIG_JAC_TOL2, EIG_MAX_SWEEPS, capped, nrot);
    double lx = 0.0, ly = 0.0;
#pragma unroll
    for (int i = 0; i < RL; ++i) {
        lx = fma(x[i], x[i], lx);
        ly = fma(y[i], y[i], ly);
    }
    lx = sum8(lx);
    ly = sum8(ly);
    if (r == 0 && g < G) {
        sh.key[2 * g] = rankable(ly);
        sh.key[2 * g + 1] = rankable(lx);
    }
    __syncthreads();
    if (g < G) {
        // descending order, ties by position (an odd n's empty column ranks last)
        const int rx = (int)sum8((double)entries_before(sh.key, 2 * G, 2 * g + 1, r, 8));
        const int ry = (int)sum8((double)entries_before(sh.key, 2 * G, 2 * g, r, 8));
        const double ix = lx > 0.0 ? 1.0 / sqrt(lx) : 0.0, iy = ly > 0.0 ? 1.0 / sqrt(ly) : 0.0;
        if (r == 0) {
            if (rx < n) theta[rx] = lx - mu;
            if (ry < n) theta[ry] = ly - mu;
        }
#pragma unroll
        for (int i = 0; i < RL; ++i) {
            const int row = r + 8 * i;
            if (row < n) {
                const long o = (long)place[row] * n;
                if (rx < n) S[o + rx] = x[i] * ix;
                if (ry < n) S[o + ry] = y[i] * iy;
            }
        }
    }
    if (tid == 0) {
        ctl->sweeps = (rounds + 2 * G - 1) / (2 * G);
        ctl->jac_capped = capped ? 1 : 0;
    }
}

template <int NF>
static void launch_dense(const double* E, int n, const EigWork& w, hipStream_t stream) {
    hipLaunchKernelGGL((eig_dense_kernel<NF>), dim3(1), dim3(64 * NF), 0, stream, E, n, w.theta, w.S, w.ctl);
}

// ---------------------------------------------------------------- factor of the Gram matrix

// norm[i] = |Y_i| (0 for a vanishing column) and the factor L of the scaled
// Gram matrix (unit diagonal) in sh.buf.
template <int NF>
__device__ __forceinline__ void factor_gram(const double* __restrict__ Gt, SmallEig<NF>& sh, double* norm) {
    using Sh = SmallEig<NF>;
    constexpr int P = Sh::P, LDA = Sh::LDA;
    const int tid = threadIdx.x;
    for (int i = tid; i < P; i += 64 * NF) {
        const double g = Gt[gram_tile(NF, i >> 4, i >> 4) * 256 + (i & 15) * 17];
        norm[i] = g > 1e-280 ? sqrt(g) : 0.0;
    }
    __syncthreads();
    for (int attempt = 0;; ++attempt) {
        for (int e = tid; e < P * P; e += 64 * NF) {
            const int i = e / P, j = e - (e / P) * P;
            if (j > i) continue;
            const double dd = norm[i] * norm[j];
            double v = i == j ? 1.0 : 0.0;
            if (dd > 0.0 && i != j) v = Gt[gram_tile(NF, j >> 4, i >> 4) * 256 + (j & 15) * 16 + (i & 15)] / dd;
            if (i == j && attempt) v += EIG_SHIFT;
            sh.buf[i * LDA + j] = v;
            if ((i >> 4) == (j >> 4)) sh.buf[j * LDA + i] = v;   // diagonal blocks whole
        }
        __syncthreads();
        chol_blocked<NF>(sh.buf, 0.1 * EIG_SHIFT, sh.linv, &sh.minp);
        const bool good = attempt || sh.minp >= EIG_PIV_OK;
        __syncthreads();
        if (good) break;
    }
}

// Power pass: Q = D L^-T (upper triangular, row-major), so that Z Q has
// orthonormal columns.  The inverse by 16 x 16 blocks: the diagonal ones by
// substitution, one lane a row, then wave i the block row i on the matrix
// cores (a product's result registers are the next one's operand).
// CholeskyQR's one-workgroup part; the unblocked kernel before it (one
// barrier a column) took 34 / 72 us at p = 48 / 80; this takes 18 / 38 us.
template <int NF>
__global__ __launch_bounds__(64 * NF) void eig_power_kernel(const double* __restrict__ Gt, int n,
                                                            double* __restrict__ Q, double* __restrict__ dout,
                                                            const EigCtl* ctl) {
    if (eig_done(ctl)) return;
    using Sh = SmallEig<NF>;
    constexpr int P = Sh::P, LDA = Sh::LDA;
    __shared__ Sh sh;
    __shared__ double norm[P];
    __shared__ double xd[NF][16][17];   // inverses of the diagonal blocks
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 15, fk = lane >> 4;
    factor_gram<NF>(Gt, sh, norm);
    {
        // row fr of the inverse of diagonal block `wave` (all four lane
        // groups the same, group 0 stores)
        const double* Lb = sh.buf + 16 * wave * LDA + 16 * wave;
        double x[16];
#pragma unroll
        for (int i = 15; i >= 0; --i) {
            double v = i == fr ? 1.0 : 0.0;
#pragma unroll
            for (int m = 15; m > i; --m) v = fma(-Lb[m * LDA + i], x[m], v);
            x[i] = v * sh.linv[16 * wave + i];
            if (fk == 0) xd[wave][fr][i] = x[i];
        }
    }
    __syncthreads();
    // Block row i = wave of X = L^-1, as its transpose Y_j = X_ij^T, j = i .. 0:
    //   Y_j = -X_jj^T sum_{j < k <= i} L_kj^T Y_k
    // (row by row: X L = I holds to rounding, which is what Z D L^-T needs to
    // be orthonormal where L is nearly singular; solved by columns, L X = I
    // would)
    const int i = wave;
    d4 Yb[NF];
#pragma unroll
    for (int j = NF - 1; j >= 0; --j) {
        if (j > i) continue;
        if (j == i) {
#pragma unroll
            for (int q = 0; q < 4; ++q) Yb[j][q] = xd[j][fr][fk + 4 * q];
        } else {
            d4 t = d4{0, 0, 0, 0};
#pragma unroll
            for (int k = NF - 1; k > j; --k) {
                if (k > i) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    t = __builtin_amdgcn_mfma_f64_16x16x4f64(sh.buf[(16 * k + fk + 4 * q) * LDA + 16 * j + fr],
                                                             Yb[k][q], t, 0, 0, 0);
            }
            d4 o = d4{0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                o = __builtin_amdgcn_mfma_f64_16x16x4f64(-xd[j][fk + 4 * q][fr], t[q], o, 0, 0, 0);
            Yb[j] = o;
        }
        // Q[r][c] = d_r (L^-1)[c][r]; a vanishing column is replaced by
        // uniform(-1, 1) entries, of norm about sqrt(n / 3)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double nr = norm[16 * j + fk + 4 * q];
            const double dr = nr > 0.0 ? 1.0 / nr : 1.0 / sqrt(n / 3.0);
            Q[(long)(16 * j + fk + 4 * q) * P + 16 * i + fr] = dr * Yb[j][q];
        }
    }
    for (int i = tid; i < P; i += 64 * NF) dout[i] = norm[i];
}

// Ritz pass: S (row-major p x p, orthonormal columns) and theta = sigma,
// descending, of W = E V from the factor of its Gram matrix (see the top).
// One workgroup, bound by the Jacobi rounds' dependent chain (jacobi.h); the
// two-sided Jacobi of V^T W it replaces moved two matrices through LDS every
// round with two barriers, and needed the Cholesky of W^T W besides: 139 + 34
// us at p = 48, 396 + 72 us at p = 80; this takes 80 / 250 us.
template <int NF>
__global__ __launch_bounds__(64 * NF) void eig_ritz_kernel(const double* __restrict__ Gt, double* __restrict__ theta,
                                                           double* __restrict__ S, EigCtl* ctl) {
    if (eig_done(ctl)) return;
    using Sh = SmallEig<NF>;
    constexpr int P = Sh::P, LDA = Sh::LDA, RL = 2 * NF;
    __shared__ Sh sh;
    __shared__ double norm[P];
    const int tid = threadIdx.x, g = tid >> 3, r = tid & 7;
    factor_gram<NF>(Gt, sh, norm);
    double x[RL], y[RL];
#pragma unroll
    for (int i = 0; i < RL; ++i) {
        const int row = r + 8 * i, c = 2 * g;
        const double w = norm[row] > 0.0 ? norm[row] : 1e-150;
        y[i] = c <= row ? sh.buf[row * LDA + c] * w : 0.0;
        x[i] = c + 1 <= row ? sh.buf[row * LDA + c + 1] * w : 0.0;
    }
    if (tid < 2) sh.flag[tid] = -1;
    __syncthreads();
    bool capped;
    unsigned nrot = 0;
    const JacobiShared js{sh.buf, sh.nrm, sh.flag, Sh::SLOT};
    const int rounds = jacobi_rounds<RL, false>(x, y, js, Sh::G, g, r, EIG_JAC_TOL2, EIG_MAX_SWEEPS, capped, nrot);
    double lx = 0.0, ly = 0.0;
#pragma unroll
    for (int i = 0; i < RL; ++i) {
        lx = fma(x[i], x[i], lx);
        ly = fma(y[i], y[i], ly);
    }
    lx = sum8(lx);
    ly = sum8(ly);
    if (r == 0) {
        sh.key[2 * g] = rankable(ly);
        sh.key[2 * g + 1] = rankable(lx);
    }
    __syncthreads();
    // descending order, ties by position
    const int rx = (int)sum8((double)entries_before(sh.key, P, 2 * g + 1, r, 8));
    const int ry = (int)sum8((double)entries_before(sh.key, P, 2 * g, r, 8));
    const double sx = sqrt(lx), sy = sqrt(ly);
    if (r == 0) {   // a vanishing column of W: sigma 0, S its unit vector; a NaN stays one
        theta[rx] = sx <= 1e-140 ? 0.0 : sx;
        theta[ry] = sy <= 1e-140 ? 0.0 : sy;
    }
    const double ix = 1.0 / sx, iy = 1.0 / sy;
#pragma unroll
    for (int i = 0; i < RL; ++i) {
        S[(long)(r + 8 * i) * P + rx] = x[i] * ix;
        S[(long)(r + 8 * i) * P + ry] = y[i] * iy;
    }
    if (tid == 0) {
        ctl->sweeps = (rounds + P - 1) / P;
        ctl->jac_capped = capped ? 1 : 0;
    }
}

// ---------------------------------------------------------------- block products

// 16 rows of an n x p block in LDS, zeros past n
template <int NF, typename Fill>
__device__ __forceinline__ void stage_rows(double (*dst)[16 * NF + 2], const double* src, long r0, int n, Fill fill) {
    constexpr int P = 16 * NF;
    for (int e = threadIdx.x; e < EIG_ROWS * P; e += 64 * NF) {
        const int r = e / P, c = e - (e / P) * P;
        dst[r][c] = r0 + r < n ? fill(src, r0 + r, c) : 0.0;
    }
}

// Power pass: V = Z Q (Q upper triangular), 16 rows a workgroup, one 16-wide
// column tile a wave.  A column of Z with norm 0 is replaced by random
// entries.  Z may be V (a workgroup stages its rows before it writes them).
template <int NF>
__global__ __launch_bounds__(64 * NF) void eig_orth_kernel(const double* Z, double* V, int n,
                                                           const double* __restrict__ Q,
                                                           const double* __restrict__ norm, unsigned long long seed,
                                                           const EigCtl* ctl) {
    if (eig_done(ctl)) return;
    constexpr int P = 16 * NF;
    __shared__ double zs[EIG_ROWS][P + 2];
    const int lane = threadIdx.x & 63, f = threadIdx.x >> 6, fr = lane & 15, fk = lane >> 4;
    const long r0 = (long)blockIdx.x * EIG_ROWS;
    stage_rows<NF>(zs, Z, r0, n, [&](const double* src, long r, int c) {
        return norm[c] > 0.0 ? src[r * P + c]
                             : hash_uniform(seed ^ (0xD1B54A32D192ED03ull * (unsigned long long)(r * P + c + 1)));
    });
    __syncthreads();
    d4 acc = d4{0, 0, 0, 0};
    for (int kt = 0; kt <= f; ++kt) {
        double b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = Q[(long)(16 * kt + fk + 4 * q) * P + 16 * f + fr];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(zs[fr][16 * kt + fk + 4 * q], b[q], acc, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (r0 + fk + 4 * q < n) V[(r0 + fk + 4 * q) * P + 16 * f + fr] = acc[q];
}

// Ritz pass: u = Vin S to V, E u = Win S; the next power pass's block to X
// (E u / sigma, or u where sigma is too small for it), and the workgroup's
// parts of |E u_j - sigma_j u_j|^2, |E u_j + sigma_j u_j|^2 (the eigenvalue's
// sign is the one with the smaller residual) and |u_j|^2 to rpart.  Vin and Win may be V and X (a
// workgroup stages its rows before it writes them).
template <int NF>
__global__ __launch_bounds__(64 * NF) void eig_ritz_apply_kernel(const double* Vin, const double* Win, double* V,
                                                                 double* X, int n, const double* __restrict__ S,
                                                                 const double* __restrict__ theta,
                                                                 double* __restrict__ rpart, const EigCtl* ctl) {
    if (eig_done(ctl)) return;
    constexpr int P = 16 * NF;
    __shared__ double vs[EIG_ROWS][P + 2];
    __shared__ double ws[EIG_ROWS][P + 2];
    const int lane = threadIdx.x & 63, f = threadIdx.x >> 6, fr = lane & 15, fk = lane >> 4;
    const long r0 = (long)blockIdx.x * EIG_ROWS;
    auto plain = [&](const double* src, long r, int c) { return src[r * P + c]; };
    stage_rows<NF>(vs, Vin, r0, n, plain);
    stage_rows<NF>(ws, Win, r0, n, plain);
    const double sig = theta[16 * f + fr], top = theta[0];
    __syncthreads();
    d4 au = d4{0, 0, 0, 0}, aw = d4{0, 0, 0, 0};
#pragma unroll
    for (int kt = 0; kt < NF; ++kt) {
        double b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = S[(long)(16 * kt + fk + 4 * q) * P + 16 * f + fr];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            au = __builtin_amdgcn_mfma_f64_16x16x4f64(vs[fr][16 * kt + fk + 4 * q], b[q], au, 0, 0, 0);
            aw = __builtin_amdgcn_mfma_f64_16x16x4f64(ws[fr][16 * kt + fk + 4 * q], b[q], aw, 0, 0, 0);
        }
    }
    const bool advance = sig > EIG_ADVANCE * top;
    const double inv = advance ? 1.0 / sig : 0.0;
    double res = 0.0, neg = 0.0, len = 0.0;   // rows past n are zero in both factors
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double d = fma(-sig, au[q], aw[q]), e = fma(sig, au[q], aw[q]);
        res = fma(d, d, res);
        neg = fma(e, e, neg);
        len = fma(au[q], au[q], len);
        const long row = r0 + fk + 4 * q;
        if (row < n) {
            V[row * P + 16 * f + fr] = au[q];
            X[row * P + 16 * f + fr] = advance ? aw[q] * inv : au[q];
        }
    }
    res += __shfl_xor(res, 16, 64);
    res += __shfl_xor(res, 32, 64);
    neg += __shfl_xor(neg, 16, 64);
    neg += __shfl_xor(neg, 32, 64);
    len += __shfl_xor(len, 16, 64);
    len += __shfl_xor(len, 32, 64);
    if (fk == 0) {
        double* out = rpart + (long)blockIdx.x * (3 * EIG_PMAX) + 16 * f + fr;
        out[0] = res;
        out[EIG_PMAX] = neg;
        out[2 * EIG_PMAX] = len;
    }
}

// After a Ritz pass: the residuals summed over the workgroups' parts (fixed
// order), the eigenvalues with their signs in descending order (lam, and ord:
// the column of V of each; an E computed in a split precision has small
// negative ones, which rank last although the block finds them by size),
// whether the solve stops here, and unit: the factor that makes u_j a unit
// vector.  One CholeskyQR leaves a column with pivot d orthogonal to
// eps / sqrt(d) but its length to eps / d only; pivots are small where a kept
// block meets an environment that has moved (3e-11 of length and 4e-14 of angle
// at T = 1.9, D = 48) or columns are rounding noise.  A length within 1e-12
// stays as it is.
__global__ __launch_bounds__(768) void eig_check_kernel(const double* __restrict__ rpart, int nb, int p, int k,
                                                        const double* __restrict__ theta, double* __restrict__ lam,
                                                        int* __restrict__ ord, double* __restrict__ unit,
                                                        double mu_rel, double tol, int it, int last_iter,
                                                        EigCtl* ctl) {
    if (eig_done(ctl)) return;
    __shared__ double sh[8][EIG_PMAX], sn[8][EIG_PMAX], sl[8][EIG_PMAX];
    __shared__ double th[EIG_PMAX];
    __shared__ double top;
    const int j = threadIdx.x % EIG_PMAX, seg = threadIdx.x / EIG_PMAX;
    double s = 0.0, m = 0.0, len = 0.0;
    if (j < p)
#pragma unroll 4
        for (int b = seg; b < nb; b += 8) {
            const double* part = rpart + (long)b * (3 * EIG_PMAX) + j;
            s += part[0];
            m += part[EIG_PMAX];
            len += part[2 * EIG_PMAX];
        }
    sh[seg][j] = s;
    sn[seg][j] = m;
    sl[seg][j] = len;
    __syncthreads();
    double mine = 0.0;
    if (seg == 0) {
#pragma unroll
        for (int i = 1; i < 8; ++i) {
            s += sh[i][j];
            m += sn[i][j];
            len += sl[i][j];
        }
        if (j < p) unit[j] = fabs(len - 1.0) > 1e-12 && len > 0.0 ? 1.0 / sqrt(len) : 1.0;
        mine = j < p ? (m < s ? -theta[j] : theta[j]) : -INFINITY;
        th[j] = rankable(mine);
    }
    __syncthreads();
    if (seg == 0) {
        // a permutation of the columns, also where values are NaN: eig_select
        // reads ord as column numbers
        const int rk = descending_place(th, EIG_PMAX, j);
        if (j < p) {
            lam[rk] = mine - mu_rel * ctl->trace;
            ord[rk] = j;
        }
        if (rk == 0) top = mine;
        sh[0][j] = j < p && rk < k ? fmin(s, m) : 0.0;
    }
    __syncthreads();
    if (threadIdx.x < 32) sh[0][j] = fmax(sh[0][j], fmax(sh[0][j + 32], sh[0][j + 64]));
    __syncthreads();
    for (int h = 16; h > 0; h >>= 1) {
        if (threadIdx.x < h) sh[0][j] = fmax(sh[0][j], sh[0][j + h]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double worst = sqrt(fmax(sh[0][0], 0.0));
        const double scale = fmax(fabs(top), 1e-300);
        const int conv = worst <= tol * scale;
        const double res = worst / scale;
        ctl->iters = it + 1;
        ctl->resid = res;
        ctl->converged = conv;
        // stagnation: three checks in a row without getting below 0.9x
        // the best residual so far mean the block has reached its
        // rounding floor (kept pairs in the noise of a nearly rank-
        // deficient E); further passes would end at the same residual at
        // the pass cap, so stop here (converged stays 0, as at the cap)
        if (res < 0.9 * ctl->best) {
            ctl->best = res;
            ctl->stall = 0;
        } else {
            ctl->stall += 1;
        }
        if (conv || it == last_iter || ctl->stall >= 3) ctl->done = 1;
    }
}

// ---------------------------------------------------------------- output

// Columns ord[0], ord[1], ... (or 0, 1, ...) of the row-major n x ldv block Vr,
// times their factors in unit (none: 1): largest-magnitude entry made positive
// (lowest index on ties), written as Ut[l, i] = u_l[i] and
// Ux[l, a2, a1] = u_l[a1 * dx + a2].
__device__ __forceinline__ void put_val(const Buf& o, size_t idx, double v) {
    switch (o.fmt) {
        case Fmt::F64: static_cast<double*>(o.ptr)[idx] = v; break;
        case Fmt::F32: static_cast<float*>(o.ptr)[idx] = (float)v; break;
        default: {
            __bf16* q = static_cast<__bf16*>(o.ptr);
            const float f = (float)v;
            const __bf16 h = (__bf16)f;
            q[idx] = h;
            const float r = f - (float)h;
            const __bf16 m = (__bf16)r;
            q[idx + o.plane] = m;
            if (o.fmt == Fmt::BF16x3) q[idx + 2 * o.plane] = (__bf16)(r - (float)m);
        }
    }
}

// One block per kept column l.
__global__ __launch_bounds__(256) void eig_select_kernel(const double* __restrict__ Vr, const int* __restrict__ ord,
                                                         const double* __restrict__ unit, int ldv, int n, int dx,
                                                         Buf Ut, Buf Ux) {
    __shared__ double sv[256];
    __shared__ int si[256];
    const int l = blockIdx.x;
    const int col = ord ? ord[l] : l;
    Vr += col;
    Entry e = largest_entry(Vr, ldv, n, threadIdx.x, 256);
    sv[threadIdx.x] = e.size;
    si[threadIdx.x] = e.row;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            e = larger_entry(e, Entry{sv[threadIdx.x + s], si[threadIdx.x + s]});
            sv[threadIdx.x] = e.size;
            si[threadIdx.x] = e.row;
        }
        __syncthreads();
    }
    const double len = unit ? unit[col] : 1.0;
    const double sgn = Vr[(long)si[0] * ldv] < 0.0 ? -len : len;
    for (int i = threadIdx.x; i < n; i += 256) {
        const double u = sgn * Vr[(long)i * ldv];
        put_val(Ut, (size_t)l * n + i, u);
        const int a1 = i / dx, a2 = i - (i / dx) * dx;
        put_val(Ux, ((size_t)l * dx + a2) * dx + a1, u);
    }
}

__global__ __launch_bounds__(64) void eig_stats_kernel(const double* __restrict__ theta, int p, int n, int k,
                                                       const EigCtl* ctl, DevState* st, int step, int slot,
                                                       double fail_tol) {
    if (threadIdx.x != 0 || step >= 64) return;
    // how the solve ended, and whether it failed: a dense diagonalisation
    // (p == n) fails only at its sweep cap; a subspace solve that stopped
    // short of the convergence bound fails when its residual is above
    // fail_tol (NaN included); non-finite eigenvalues fail either way
    int stop;
    bool failed;
    if (p == n) {
        stop = ctl->jac_capped ? HOTRG_EIG_PASS_CAP : HOTRG_EIG_CONVERGED;
        failed = ctl->jac_capped != 0;
    } else {
        stop = ctl->converged ? HOTRG_EIG_CONVERGED : (ctl->stall >= 3 ? HOTRG_EIG_STAGNATED : HOTRG_EIG_PASS_CAP);
        failed = !ctl->converged && !(ctl->resid <= fail_tol);
    }
    if (!isfinite(theta[0]) || !isfinite(ctl->trace)) failed = true;
    if (failed && st->status == 0) st->status = HOTRG_EEIG;
    double err;
    if (p == n) {   // every eigenvalue known: discarded weight summed directly
        double tot = 0.0, dis = 0.0;
        for (int j = 0; j < n; ++j) {
            tot += theta[j];
            if (j >= k) dis += theta[j];
        }
        err = tot != 0.0 ? dis / tot : 0.0;
    } else {
        double kept = 0.0;
        for (int j = 0; j < k; ++j) kept += theta[j];
        const double tr = ctl->trace;
        err = tr != 0.0 ? (tr - kept) / tr : 0.0;
    }
    const double gap = k < n ? (k < p ? (theta[k - 1] - theta[k]) / theta[0] : NAN) : INFINITY;
    if (slot == 0) {
        st->trunc_err[step] = err;
        st->eps_left[step] = err;
        st->cut_gap[step] = gap;
        st->info[step] = ctl->iters;
        st->eig_resid[step] = ctl->resid;
        st->eig_sweeps[step] = ctl->sweeps;
        st->eig_stop[step] = stop;
        st->side[step] = 0;
    } else {
        st->eps_right[step] = err;
        st->r_cut_gap[step] = gap;
        st->r_info[step] = ctl->iters;
        st->r_resid[step] = ctl->resid;
        st->r_sweeps[step] = ctl->sweeps;
        st->r_eig_stop[step] = stop;
    }
}

// Two-sided truncation (the side with the smaller discarded weight wins,
// ties keep the left one).  Every block reads the same two numbers, so all
// take the same branch; block 0 records the outcome.
__global__ __launch_bounds__(256) void choose_side_kernel(DevState* st, int step, uint4* __restrict__ Ut,
                                                          uint4* __restrict__ Ux, const uint4* __restrict__ UtR,
                                                          const uint4* __restrict__ UxR, size_t words) {
    if (step >= 64) return;
    const bool right = st->eps_right[step] < st->eps_left[step];
    if (right) {
        for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < words; i += (size_t)gridDim.x * 256) {
            Ut[i] = UtR[i];
            Ux[i] = UxR[i];
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->side[step] = right ? 1 : 0;
        if (right) {
            st->trunc_err[step] = st->eps_right[step];
            st->cut_gap[step] = st->r_cut_gap[step];
            st->info[step] = st->r_info[step];
            st->eig_resid[step] = st->r_resid[step];
            st->eig_sweeps[step] = st->r_sweeps[step];
            st->eig_stop[step] = st->r_eig_stop[step];
        }
    }
}

// ---------------------------------------------------------------- host side

static unsigned grid_for(long count, int per) { return (unsigned)((count + per - 1) / per); }

// One thread copies the eigensolve's stop state to host memory as one
// system-scope store, so that the host sees it without a copy engine or an
// event.
__global__ __launch_bounds__(64) void eig_mail_kernel(const EigCtl* __restrict__ ctl, EigMail* mail, int seq) {
    if (threadIdx.x != 0) return;
    const unsigned long long word = ((unsigned long long)(unsigned)seq << 32) |
                                    ((unsigned long long)(unsigned)ctl->iters << 1) | (ctl->done ? 1ull : 0ull);
    __hip_atomic_store(&mail->word, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_eig_mail(const EigCtl* ctl, EigMail* mail, int seq, hipStream_t stream) {
    hipLaunchKernelGGL(eig_mail_kernel, dim3(1), dim3(64), 0, stream, ctl, mail, seq);
    return hipGetLastError();
}

hipError_t launch_choose_side(DevState* st, int step, void* Ut, void* Ux, const void* UtR, const void* UxR,
                              size_t bytes, hipStream_t stream) {
    if (bytes % 16) return hipErrorInvalidValue;
    const size_t words = bytes / 16;
    unsigned blocks = grid_for((long)words, 256);
    if (blocks > 1024) blocks = 1024;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(choose_side_kernel, dim3(blocks), dim3(256), 0, stream, st, step, static_cast<uint4*>(Ut),
                       static_cast<uint4*>(Ux), static_cast<const uint4*>(UtR), static_cast<const uint4*>(UxR), words);
    return hipGetLastError();
}

// One pass of the subspace iteration.  A power pass reads the block the last
// Ritz pass left in w.W (the first one V itself) and writes V; a Ritz pass
// reads V, whose columns the power pass before it made orthonormal: the Ritz
// vectors are as orthonormal as the block they are formed from.  The last pass
// of an odd limit follows no power pass (it reads what a power pass would), and
// makes its block orthonormal itself, twice, since that block may be anything.
template <int NF>
static void launch_pass(const double* E, int n, int k, const EigWork& w, double* V, int it, int maxit, bool ritz,
                        double mu, bool twice, double tol, unsigned long long seed, hipStream_t stream) {
    const int nb = (n + EIG_ROWS - 1) / EIG_ROWS;
    const int count = gram_tiles(NF) * 256;
    const bool after_power = it % EIG_RR_EVERY != 0;
    auto sum_gram = [&] {
        hipLaunchKernelGGL(eig_sum_kernel, dim3(count / 32), dim3(256), 0, stream, w.part, nb, count, w.G, w.ctl);
    };
    // V = src Q from the Gram parts of src
    auto apply_factor = [&](const double* src) {
        sum_gram();
        hipLaunchKernelGGL((eig_power_kernel<NF>), dim3(1), dim3(64 * NF), 0, stream, w.G, n, w.S, w.dsc, w.ctl);
        hipLaunchKernelGGL((eig_orth_kernel<NF>), dim3(nb), dim3(64 * NF), 0, stream, src, V, n, w.S, w.dsc,
                           seed * 131 + it, w.ctl);
    };
    auto orthonormalise = [&](const double* src) {
        hipLaunchKernelGGL((eig_gram_kernel<NF>), dim3(nb), dim3(64 * NF), 0, stream, src, n, w.part, w.ctl);
        apply_factor(src);
    };
    const double* in = it == 0 || after_power ? V : w.W;
    double* out = after_power ? w.W : w.Z;
    if (ritz && !after_power) {
        orthonormalise(in);
        orthonormalise(V);
        in = V;
    }
    hipLaunchKernelGGL((eig_ev_kernel<NF>), dim3(nb), dim3(512), 0, stream, E, n, in, out, w.part,
                       mu, w.ctl);
    if (!ritz) {
        apply_factor(out);
        if (twice) orthonormalise(V);
        return;
    }
    sum_gram();
    hipLaunchKernelGGL((eig_ritz_kernel<NF>), dim3(1), dim3(64 * NF), 0, stream, w.G, w.theta, w.S, w.ctl);
    hipLaunchKernelGGL((eig_ritz_apply_kernel<NF>), dim3(nb), dim3(64 * NF), 0, stream, in, out, V, w.W, n, w.S,
                       w.theta, w.rpart, w.ctl);
    hipLaunchKernelGGL(eig_check_kernel, dim3(1), dim3(768), 0, stream, w.rpart, nb, 16 * NF, k, w.theta,
                       w.lam, w.ord, w.dsc, mu, tol, it, maxit - 1, w.ctl);
}

hipError_t launch_eig_topk(const double* E, int n, int k, int dx, const EigWork& w, int parity, bool warm,
                           unsigned long long seed, int maxit, double tol, double fail_tol, const Buf& Ut,
                           const Buf& Ux, DevState* st, int step, hipStream_t stream, bool renew, int slot,
                           const EigRange& range) {
    if (n < 1 || k < 1 || k > n || maxit < 1) return hipErrorInvalidValue;
    const int it_first = range.first < 0 ? 0 : range.first;
    const int it_last = range.last < 0 || range.last > maxit ? maxit : range.last;
    if (n <= EIG_PMAX) {
        if (!range.start) return hipSuccess;
        hipLaunchKernelGGL(eig_init_kernel, dim3(1), dim3(256), 0, stream, E, n, (double*)nullptr, 0, 1, seed, w.ctl);
        switch ((n + 15) / 16) {
            case 1: launch_dense<1>(E, n, w, stream); break;
            case 2: launch_dense<2>(E, n, w, stream); break;
            case 3: launch_dense<3>(E, n, w, stream); break;
            case 4: launch_dense<4>(E, n, w, stream); break;
            case 5: launch_dense<5>(E, n, w, stream); break;
            default: launch_dense<6>(E, n, w, stream); break;
        }
        hipLaunchKernelGGL(eig_select_kernel, dim3(k), dim3(256), 0, stream, w.S,
                           (const int*)nullptr, (const double*)nullptr, n, n, dx, Ut, Ux);
        hipLaunchKernelGGL(eig_stats_kernel, dim3(1), dim3(64), 0, stream, w.theta, n, n, k, w.ctl, st, step, slot,
                           fail_tol);
        return hipGetLastError();
    }
    const int p = eig_block(n, k);
    if (p <= k || p % 16 || p < 32 || p > EIG_PMAX) return hipErrorInvalidValue;
    double* V = w.V[parity];
    const unsigned g_init = grid_for((long)n * p, 256) > 1024 ? 1024 : grid_for((long)n * p, 256);
    if (range.start)
        hipLaunchKernelGGL(eig_init_kernel, dim3(g_init), dim3(256), 0, stream, E, n, V, p, warm ? 1 : 0, seed,
                           w.ctl);
    // warm: E + mu I in place of E (the same eigenvectors), mu far below the
    // convergence bound: a column of the block in the rounding noise of E
    // keeps its direction instead of taking that of the noise, which has
    // fewer dimensions than such columns (it follows the rows of E).  A cold
    // block has no direction worth keeping; `renew` orthonormalises it twice.
    const double mu = warm ? EIG_MU : 0.0;
    const bool twice = renew && !warm;
    for (int it = it_first; it < it_last; ++it) {
        const bool ritz = it % EIG_RR_EVERY == EIG_RR_EVERY - 1 || it == maxit - 1;
        switch (p / 16) {
            case 2: launch_pass<2>(E, n, k, w, V, it, maxit, ritz, mu, twice, tol, seed, stream); break;
            case 3: launch_pass<3>(E, n, k, w, V, it, maxit, ritz, mu, twice, tol, seed, stream); break;
            case 4: launch_pass<4>(E, n, k, w, V, it, maxit, ritz, mu, twice, tol, seed, stream); break;
            case 5: launch_pass<5>(E, n, k, w, V, it, maxit, ritz, mu, twice, tol, seed, stream); break;
            default: launch_pass<6>(E, n, k, w, V, it, maxit, ritz, mu, twice, tol, seed, stream); break;
        }
    }
    if (!range.end) return hipGetLastError();
    hipLaunchKernelGGL(eig_select_kernel, dim3(k), dim3(256), 0, stream, V, w.ord, w.dsc, p, n, dx, Ut,
                       Ux);
    hipLaunchKernelGGL(eig_stats_kernel, dim3(1), dim3(64), 0, stream, w.lam, p, n, k, w.ctl, st, step, slot,
                       fail_tol);
    return hipGetLastError();
}

}  // namespace hotrg

// One-sided Jacobi on the columns of a small matrix, one workgroup: the
// shared rounds of the eigensolver's and (same lane helpers) the iTEBD
// update's decompositions.
//
// Columns sit on a line of 2 G positions, two of them in the registers of
// each group of eight lanes (lane r of a group holds rows r, r + 8, ...).
// Even rounds pair positions (2g, 2g + 1), odd rounds (2g + 1, 2g + 2), and
// the two columns of a pair change places after their rotation (odd-even
// ordering): every pair of columns meets exactly once in 2 G consecutive
// rounds.  With the exchange a column stays in a group for two rounds and
// then moves to a neighbour, so a round passes one column per group through
// LDS (a mailbox per group, two buffers in turn) instead of reading and
// writing both, has one barrier, and needs no index arithmetic.
//
// What bounds a round is its dependent chain: mailbox read, the pair's dot
// product over eight lanes (three DPP stages), the rotation's angle, the
// rotation, mailbox write, barrier (0.27 us with 3 rows a lane, 0.43 with 8;
// four lanes a pair, which halves the waves that pay for the angle, was 20%
// slower with two workgroups on a CU).  The squared norms travel with the
// columns (updated by the rotation, recomputed once per sweep), so a round
// forms one dot product instead of three, and the angle comes from two
// reciprocal square roots refined from the hardware estimate instead of
// IEEE divisions and square roots.
#pragma once

#include <hip/hip_runtime.h>

#include "jacobi_rule.h"

namespace hotrg {

// a double from another lane of the same row through a DPP move of each half
template <int Ctrl>
__device__ __forceinline__ double dpp_d(double v) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, Ctrl, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), Ctrl, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// sum over an aligned group of eight lanes: partner lane ^1 (quad_perm
// [1,0,3,2]), ^2 (quad_perm [2,3,0,1]), then the mirror lane 7 - l inside
// the half-row (the other quad); every lane gets the same bits
__device__ __forceinline__ double sum8(double v) {
    v += dpp_d<0xB1>(v);
    v += dpp_d<0x4E>(v);
    v += dpp_d<0x141>(v);
    return v;
}

// a double of lane l (uniform l) in every lane
__device__ __forceinline__ double readlane_d(double v, int l) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(unsigned)u, l);
    const int hi = __builtin_amdgcn_readlane((int)(unsigned)(u >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// largest value over the 64 lanes of a wave, in every lane
__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp_d<0xB1>(v));
    v = fmax(v, dpp_d<0x4E>(v));
    v = fmax(v, dpp_d<0x141>(v));
    v = fmax(v, dpp_d<0x140>(v));
    return fmax(fmax(readlane_d(v, 0), readlane_d(v, 16)), fmax(readlane_d(v, 32), readlane_d(v, 48)));
}

// 1 / x, x > 0 normal: the hardware estimate (2^-24) and one third-order step
__device__ __forceinline__ double rcp_nr(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y * e, 1.0 + e, y);
}

// 1 / sqrt(x), x > 0 finite: the hardware estimate (relative error 2^-24
// measured on gfx950) and one third-order step, which leaves rounding errors
// only; a dependent chain of six operations
__device__ __forceinline__ double rsqrt_nr(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// The rotation that makes columns p, q orthogonal (al = p.p, be = q.q,
// ga = p.q): p' = c p - s q, q' = s p + c q, and t = s / c, by which the
// squared norms change (al - t ga, be + t ga).  With d = be - al and
// h = d^2 + 4 ga^2: c^2 = (1 + |d| / sqrt h) / 2, s = sign(d) ga / (c sqrt h)
// (the smaller of the two angles).  h > 0 whenever the pair passes its
// rotation test.
__device__ __forceinline__ void jacobi_angle(double al, double be, double ga, double& c, double& s, double& t) {
    const double d = be - al;
    const double h = fma(d, d, 4.0 * (ga * ga));
    const double y = rsqrt_nr(h);
    const double c2 = fma(0.5 * fabs(d), y, 0.5);
    const double w = rsqrt_nr(c2);
    c = c2 * w;
    s = (d >= 0.0 ? ga : -ga) * y * w;
    t = s * w;
}

struct JacobiShared {
    double* mail;   // [2][G][slot]: the columns in flight
    double* nrm;    // [2][G]: their squared norms
    int* flag;      // [2]: last even / odd round with a large rotation (set to -1 before the call)
    int slot;       // doubles per mailbox slot
};

// x.y over a group of eight lanes (two partial sums a lane)
template <int RL>
__device__ __forceinline__ double group_dot(const double (&x)[RL], const double (&y)[RL]) {
    double s0 = x[0] * y[0], s1 = x[1] * y[1];
#pragma unroll
    for (int i = 2; i < RL; ++i) {
        if (i & 1)
            s1 = fma(x[i], y[i], s1);
        else
            s0 = fma(x[i], y[i], s0);
    }
    return sum8(s0 + s1);
}

// Rounds until 2 G consecutive ones make no large rotation (jacobi_rule.h; pairs
// of nearly equal norms turn by large angles at any cosine and count as large),
// or max_sweeps sweeps of 2 G rounds have run.  On entry x holds the column at position 2g + 1 and y
// the one at 2g (RL rows per lane); on return the group holds two
// columns, of some order and sign.  A pair is rotated while ga^2 > tol2 al be.
// Every thread of the workgroup calls it (groups g >= G hold nothing; with
// IDLE, for workgroups that have whole waves of them, those only join the
// barriers).  Returns the rounds run; capped:
// rotations were still being made when the sweep limit ended it; nrot grows
// by the group's rotations.
template <int RL, bool IDLE>
__device__ int jacobi_rounds(double (&x)[RL], double (&y)[RL], const JacobiShared& sh, int G, int g, int r,
                             double tol2, int max_sweeps, bool& capped, unsigned& nrot) {
    const bool act = g < G;
    const bool work = !IDLE || __any(act);   // the same in every lane of a wave
    const bool last = g == G - 1;
    const int to_prev = g == 0 ? G - 1 : g - 1, to_next = last ? 0 : g + 1;
    double nx = 0.0, ny = 0.0;
    int last_rot = -1;
    const int m = 2 * G;
    const int cap = max_sweeps * m;
    int rd = 0;
    // one rotation of the pair (x, y); true in the lanes of a pair that made a large one.
    // No branch: a pair that passes no test gets the identity.  swap: x and
    // y change places instead (y negated; a column's sign is free)
    auto rotate = [&](bool on, bool swap) -> bool {
        const double ga = group_dot<RL>(x, y);
        const double ga2 = ga * ga, nn = nx * ny;
        const bool rot = on && jacobi_rotates(ga2, nn, tol2);
        double c, s, t;
        jacobi_angle(nx, ny, ga, c, s, t);
        const bool large = rot && jacobi_large(ga2, nn, s * s);
        c = rot ? c : (swap ? 0.0 : 1.0);
        s = rot ? s : (swap ? -1.0 : 0.0);
        t = rot ? t : 0.0;
#pragma unroll
        for (int i = 0; i < RL; ++i) {
            const double p = x[i], q = y[i];
            x[i] = fma(c, p, -(s * q));
            y[i] = fma(s, p, c * q);
        }
        const double ax = fma(-t, ga, nx), ay = fma(t, ga, ny);
        nrot += rot ? 1u : 0u;
        nx = swap ? ay : ax;
        ny = swap ? ax : ay;
        return large;
    };
    auto send = [&](const double (&v)[RL], double nv, int slot) {
        double* o = sh.mail + slot * sh.slot;
#pragma unroll
        for (int i = 0; i < RL; ++i) o[r + 8 * i] = v[i];
        if (r == 0) sh.nrm[slot] = nv;
    };
    auto receive = [&](double (&v)[RL], double& nv, int slot) {
        const double* o = sh.mail + slot * sh.slot;
#pragma unroll
        for (int i = 0; i < RL; ++i) v[i] = o[r + 8 * i];
        nv = sh.nrm[slot];
    };
    for (;;) {
        if (rd % m == 0 && work) {   // the norms, afresh once per sweep
            nx = group_dot<RL>(x, x);
            ny = group_dot<RL>(y, y);
        }
        // even round: x (now at position 2g) leaves to the previous group
        if (work) {
            if (rotate(act, false) && r == 0) sh.flag[0] = rd;
            if (act) send(x, nx, to_prev);
        }
        __syncthreads();
        if (act) receive(x, nx, g);
        last_rot = max(last_rot, sh.flag[0]);
        // odd round: y (now at position 2g + 2) leaves to the next group.
        // The last group holds positions 2G - 1 and 0, which are no pair: it
        // swaps its registers instead, keeps the one and sends the other back
        if (work) {
            if (rotate(act && !last, last) && r == 0) sh.flag[1] = rd + 1;
            if (act) send(y, ny, G + to_next);
        }
        __syncthreads();
        if (act) receive(y, ny, G + g);
        last_rot = max(last_rot, sh.flag[1]);
        rd += 2;
        // the flags read above are written again only after the barrier of
        // the next round of the same parity: every thread has the same last_rot
        if (rd - 1 - last_rot >= m) {
            capped = false;
            break;
        }
        if (rd >= cap) {
            capped = true;
            break;
        }
    }
    return rd;
}

}  // namespace hotrg

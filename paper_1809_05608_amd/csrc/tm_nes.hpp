// Neutrino-electron scattering sums of sixteen zones per wavefront, on the matrix cores.
//
// Lane 16 a + j holds groups a, 4 + a, 8 + a, ... of zone j: the natural order of the 4 x 4 x 4 matrix products (see
// tm_tile.hpp) with the sixteen zones as columns.  Padding groups may hold any finite value.
#pragma once

#include "tm_tile.hpp"

namespace tmk {

template <int T>
struct NesLds {
    double P[T * T * 16];          // tile (t, s) as an A operand: P[4t + b][4s + a] at 4a + b
    double near[T][6][4];          // P[k][k - n] (n = 1..3), then P[k][k + n], of row a of tile t
    // by all threads of a block; the caller synchronises
    template <int THREADS = kBlock>
    __device__ __forceinline__ void fill(const Consts& cs) {
#pragma unroll
        for (int x = threadIdx.x; x < T * T * 16; x += THREADS) {
            const int tile = x / 16, ka = (x % 16) / 4, kb = x % 4;
            P[x] = cs.P[4 * (tile / T) + kb][4 * (tile % T) + ka];
        }
        for (int x = threadIdx.x; x < T * 24; x += THREADS) {
            const int n = (x / 4) % 6, row = x % 4, k = 4 * (x / 24) + row;
            const int col = n < 3 ? row - 1 - n : row + n - 2;           // within the tile
            near[x / 24][n][row] = col >= 0 && col < 4 ? cs.P[k][k - row + col] : 0.0;
        }
    }
};

// The two NES sums of every group of 16 zones (without amp), eq. d8b with the detailed-balance factor
// exp(-|eps_k - eps_k'|/T) as a product of neighbour factors d_j = exp(-(eps_{j+1} - eps_j)/T), all at most 1:
//   sin_k  = sum_{k' > k} P psi_k'       + sum_{k' < k} P d_{k'} .. d_{k-1} psi_k'
//   sout_k = sum_{k' < k} P (1 - psi_k') + sum_{k' > k} P d_k .. d_{k'-1} (1 - psi_k').
// Between tiles of four groups the product splits into F_k (from the tile's first group to k), R_k (from k to the
// next tile's first group) and the whole tiles between, R of their first groups, applied as the sum passes them.
// Inside a tile the vector is shifted one group at a time, times d.
template <int T>
__device__ __forceinline__ void nes_sums(const NesLds<T>& sm, const double (&p)[T], const double (&d)[T], int a, int b,
                                         int ab, double (&sin_)[T], double (&sout)[T]) {
    const double to_up = a == b + 1 ? 1.0 : 0.0, to_dn = a + 1 == b ? 1.0 : 0.0;    // shift matrices, A operands
    double F[T], R[T], W[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const double d0 = mfma4(a == 0 ? 1.0 : 0.0, d[t], 0.0), d1 = mfma4(a == 1 ? 1.0 : 0.0, d[t], 0.0);
        const double d2 = mfma4(a == 2 ? 1.0 : 0.0, d[t], 0.0), d3 = mfma4(a == 3 ? 1.0 : 0.0, d[t], 0.0);
        const double lo = d0 * d1, hi = d2 * d3;
        W[t] = lo * hi;
        const double f3 = lo * d2, r1 = d1 * hi;        // both arms of every choice are at hand: no branches
        const double f01 = a == 0 ? 1.0 : d0, f23 = a == 2 ? lo : f3;
        const double r01 = a == 0 ? W[t] : r1, r23 = a == 2 ? hi : d3;
        F[t] = a < 2 ? f01 : f23;
        R[t] = a < 2 ? r01 : r23;
    }
    double dn[T], up[T];
#pragma unroll
    for (int t = 0; t < T; ++t) sin_[t] = sout[t] = dn[t] = up[t] = 0.0;
#pragma unroll
    for (int s = 0; s < T; ++s) {                       // sources below: t > s
        __builtin_amdgcn_sched_barrier(0);
        const double q = R[s] * p[s], h = 1.0 - p[s];
#pragma unroll
        for (int t = s + 1; t < T; ++t) {
            const double P = sm.P[(t * T + s) * 16 + ab];
            dn[t] = mfma4(P, q, s > 0 ? dn[t] * W[s] : 0.0);
            sout[t] = mfma4(P, h, sout[t]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = T - 1; s >= 0; --s) {                  // sources above: t < s
        __builtin_amdgcn_sched_barrier(0);
        const double h = 1.0 - p[s], q = F[s] * h;
#pragma unroll
        for (int t = s - 1; t >= 0; --t) {
            const double P = sm.P[(t * T + s) * 16 + ab];
            up[t] = mfma4(P, q, s < T - 1 ? up[t] * W[s] : 0.0);
            sin_[t] = mfma4(P, p[s], sin_[t]);
        }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {                       // inside the tile
        __builtin_amdgcn_sched_barrier(0);
        const double P = sm.P[(t * T + t) * 16 + ab], h = 1.0 - p[t];
        sin_[t] = mfma4(a > b ? P : 0.0, p[t], sin_[t]);
        sout[t] = mfma4(a < b ? P : 0.0, h, sout[t]);
        double x = F[t] * dn[t], u = p[t], y = R[t] * up[t], v = h;
#pragma unroll
        for (int n = 0; n < 3; ++n) {
            u = mfma4(to_dn, d[t] * u, 0.0);
            x = fma(sm.near[t][n][a], u, x);
            v = d[t] * mfma4(to_up, v, 0.0);
            y = fma(sm.near[t][3 + n][a], v, y);
        }
        sin_[t] += x;
        sout[t] += y;
    }
}

}  // namespace tmk

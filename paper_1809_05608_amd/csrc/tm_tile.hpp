// Dense FP64 blocks as 4 x 4 tiles on the matrix cores, four blocks per wavefront.
//
// v_mfma_f64_4x4x4 multiplies four independent pairs of 4 x 4 matrices.  With lane = 16 a + 4 g + b
// (a, b in 0..3; g the block of the wavefront) its B operand and its result hold entry (a, b) of block g's
// matrix in that lane ("natural" order), and its A operand holds entry (b, a): an A operand is the natural
// form of the transpose.  A T x T grid of tiles in natural order, one double per lane and tile, is a block of
// up to 4T rows; every product below has the A operand's transpose folded into what is stored or costs one
// more product with the identity.
//
// Vectors over the 4T rows come in three forms: "row" (lane holds element 4s + a of tile s; this is the
// B operand and the result of a matrix-vector product), "column" (element 4t + b) and "owner" (each element
// in one lane: 4b + a, and 16 + 4b + a for T > 4).
#pragma once

#include "tm_device.hpp"

namespace tmk {

__device__ __forceinline__ double mfma4(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
// c - a b (the instruction's negate bit on A)
__device__ __forceinline__ double mfma4_neg(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 1);
}

// 1/x from the hardware estimate (about 2^-22) and one cubic step: r + r (e + e^2), e = 1 - x r.
__device__ __forceinline__ double rcp_cubic(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// exp(x) for x <= 0: x = n ln 2 + r, |r| <= ln 2 / 2, Taylor series of exp(r) to r^13 (remainder below
// 2^-60) and a scale by 2^n.  The coefficients come from memory through a pointer the compiler cannot see
// through, so they are scalar operands at the point of use instead of vector registers held across a loop.
__constant__ const double kExpCoef[16] = {
    1.4426950408889634, -0x1.62e42fee00000p-1, -0x1.a39ef35793c76p-33,          // 1/ln 2, ln 2 to 32 bits, the rest of ln 2
    1.0 / 6227020800.0, 1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0, 1.0 / 362880.0, 1.0 / 40320.0,
    1.0 / 5040.0, 1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0, 0.5, 1.0};
__device__ __forceinline__ double exp_nonpos(double x) {
    typedef const __attribute__((address_space(4))) double* cptr;
    cptr c = (cptr)kExpCoef;
    asm volatile("" : "+s"(c));
    x = x > -800.0 ? x : -800.0;                   // the result is 0 from -746 on
    const double n = __builtin_rint(x * c[0]);
    const double r = fma(n, c[2], fma(n, c[1], x));
    double p = c[3];
#pragma unroll
    for (int j = 4; j < 16; ++j) p = fma(p, r, c[j]);
    return ldexp(fma(p, r, 1.0), (int)n);
}

__device__ __forceinline__ double dpp_quad(double v, int lane_of_quad) {
    const long long w = __double_as_longlong(v);
    int lo = (int)w, hi = (int)(w >> 32);
    switch (lane_of_quad) {                       // a compile-time constant after unrolling
        case 0: lo = __builtin_amdgcn_mov_dpp(lo, 0x00, 0xF, 0xF, true), hi = __builtin_amdgcn_mov_dpp(hi, 0x00, 0xF, 0xF, true); break;
        case 1: lo = __builtin_amdgcn_mov_dpp(lo, 0x55, 0xF, 0xF, true), hi = __builtin_amdgcn_mov_dpp(hi, 0x55, 0xF, 0xF, true); break;
        case 2: lo = __builtin_amdgcn_mov_dpp(lo, 0xAA, 0xF, 0xF, true), hi = __builtin_amdgcn_mov_dpp(hi, 0xAA, 0xF, 0xF, true); break;
        default: lo = __builtin_amdgcn_mov_dpp(lo, 0xFF, 0xF, 0xF, true), hi = __builtin_amdgcn_mov_dpp(hi, 0xFF, 0xF, 0xF, true); break;
    }
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

constexpr int kPivStride = 18;                    // doubles per block in the pivot exchange (16-byte aligned)

// Lane constants of the tile layout.
struct TileLane {
    int a, g, b;
    double id;                                    // identity tile
    double u0, u1, u2, u3;                        // column b of the identity
    __device__ __forceinline__ explicit TileLane(int lane) : a(lane >> 4), g((lane >> 2) & 3), b(lane & 3) {
        id = a == b ? 1.0 : 0.0;
        u0 = b == 0 ? 1.0 : 0.0;
        u1 = b == 1 ? 1.0 : 0.0;
        u2 = b == 2 ? 1.0 : 0.0;
        u3 = b == 3 ? 1.0 : 0.0;
    }
};

// Growth and zero-pivot record of an elimination: the largest multiplier magnitude (its upper word, which
// orders magnitudes to about 2^-20) and whether some 2 x 2 pivot was zero or not finite.
struct TileGuard {
    uint32_t grow = 0;
    bool zero = false;
    __device__ __forceinline__ void see(double x) { grow = max(grow, abs_key_bits(x)); }
    __device__ __forceinline__ bool tripped(double limit) const { return zero || grow > abs_key_bits(limit); }
};

// Inverse of a tile (natural in, natural out).  The sixteen entries are gathered through LDS and every lane
// solves for its own column with 2 x 2 block pivots (two reciprocals in sequence instead of four), then
// keeps its row.  The pivots are diagonal: no exchange between the two halves of the tile.
__device__ __forceinline__ double tile_inverse(double s, const TileLane& L, double* piv, TileGuard& G) {
    double* q = piv + L.g * kPivStride;
    q[4 * L.a + L.b] = s;
    wave_sync();
    const double2* v = reinterpret_cast<const double2*>(q);
    const double2 r0 = v[0], r0b = v[1], r1 = v[2], r1b = v[3], r2 = v[4], r2b = v[5], r3 = v[6], r3b = v[7];
    wave_sync();
    const double d1 = fma(r0.x, r1.y, -(r0.y * r1.x));
    const double i1 = rcp_cubic(d1);
    const double e00 = r1.y * i1, e01 = -(r0.y * i1), e10 = -(r1.x * i1), e11 = r0.x * i1;
    const double g00 = fma(r2.x, e00, r2.y * e10), g01 = fma(r2.x, e01, r2.y * e11);
    const double g10 = fma(r3.x, e00, r3.y * e10), g11 = fma(r3.x, e01, r3.y * e11);
    const double s00 = fma(-g00, r0b.x, fma(-g01, r1b.x, r2b.x)), s01 = fma(-g00, r0b.y, fma(-g01, r1b.y, r2b.y));
    const double s10 = fma(-g10, r0b.x, fma(-g11, r1b.x, r3b.x)), s11 = fma(-g10, r0b.y, fma(-g11, r1b.y, r3b.y));
    const double d2 = fma(s00, s11, -(s01 * s10));
    const double i2 = rcp_cubic(d2);
    // a zero, infinite or NaN determinant leaves a reciprocal that is not finite and non-zero
    G.zero |= !(fabs(i1) > 0.0 && fabs(i1) < INFINITY && fabs(i2) > 0.0 && fabs(i2) < INFINITY);
    // multipliers of this tile: those between the rows of the 2 x 2 pivots and those of the lower half
    G.see(r0.y * e00);
    G.see(r1.x * e00);
    G.see(g00);
    G.see(g01);
    G.see(g10);
    G.see(g11);
    G.see(s01 * (s11 * i2));
    G.see(s10 * (s11 * i2));
    const double t0 = fma(-g00, L.u0, fma(-g01, L.u1, L.u2)), t1 = fma(-g10, L.u0, fma(-g11, L.u1, L.u3));
    const double x2 = fma(s11, t0, -(s01 * t1)) * i2, x3 = fma(s00, t1, -(s10 * t0)) * i2;
    const double w0 = fma(-r0b.x, x2, fma(-r0b.y, x3, L.u0)), w1 = fma(-r1b.x, x2, fma(-r1b.y, x3, L.u1));
    const double x0 = fma(e00, w0, e01 * w1), x1 = fma(e10, w0, e11 * w1);
    const double lo = (L.a & 1) ? x1 : x0, hi = (L.a & 1) ? x3 : x2;
    return (L.a & 2) ? hi : lo;
}

// In-place inverse of a block of T x T tiles by block Gauss-Jordan with diagonal tile pivots.  For the
// M-matrices of this method (off-diagonals <= 0, columns or rows dominant) no step subtracts like-signed
// terms except on the diagonal, so entries far below the block's norm keep their relative accuracy.
template <int T>
__device__ __forceinline__ void tile_invert(double (&S)[T][T], const TileLane& L, double* piv, TileGuard& G) {
#pragma unroll
    for (int p = 0; p < T; ++p) {
        double ct[T];
#pragma unroll
        for (int i = 0; i < T; ++i)
            if (i != p) ct[i] = mfma4(S[i][p], L.id, 0.0);            // A operands of the pivot column
        const double xn = tile_inverse(S[p][p], L, piv, G);
        const double xa = mfma4(xn, L.id, 0.0);
#pragma unroll
        for (int jj = 1; jj < T; ++jj) {
            const int j = (p + jj) % T;                                // the next pivot's column first
            S[p][j] = mfma4(xa, S[p][j], 0.0);
            G.see(S[p][j]);
        }
#pragma unroll
        for (int ii = 1; ii < T; ++ii) {
            const int i = (p + ii) % T;
#pragma unroll
            for (int jj = 1; jj < T; ++jj) {
                const int j = (p + jj) % T;
                S[i][j] = mfma4_neg(ct[i], S[p][j], S[i][j]);
            }
            S[i][p] = mfma4_neg(ct[i], xn, 0.0);
        }
        S[p][p] = xn;
        asm volatile("" : "+v"(G.grow));      // keeps the record current: deferred, it would hold every step's multipliers
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Owner form of a row-form vector (element 4b + a, and 16 + 4b + a).
template <int T>
__device__ __forceinline__ void tile_row_to_owner(const double (&v)[T], const TileLane& L, double& o1, double& o2) {
    o1 = v[0];
#pragma unroll
    for (int s = 1; s < (T < 4 ? T : 4); ++s) o1 = L.b == s ? v[s] : o1;
    if constexpr (T > 4) {
        o2 = v[4];
#pragma unroll
        for (int s = 5; s < T; ++s) o2 = L.b == s - 4 ? v[s] : o2;
    }
}

}  // namespace tmk

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

// c - a b for one 16 x 16 matrix: A operand (row j, column a) and B operand (row a, column j) in lane 16 a + j,
// result row 4 r + a, column j in element r.
typedef double Vec4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ Vec4 mfma16_neg(double a, double b, Vec4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 1);
}

// 1/x from the hardware estimate (about 2^-22) and one cubic step: r + r (e + e^2), e = 1 - x r.
__device__ __forceinline__ double rcp_cubic(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// exp(x) for x <= 0: x = n ln 2 + r, |r| <= ln 2 / 2, with ln 2 in two parts whose first times n is exact (the argument
// reduction of Cody and Waite), Taylor series of exp(r) to r^13 (remainder below 2^-60) and a scale by 2^n.  The
// coefficients come from memory through a pointer the compiler cannot see through, so they are scalar operands at the
// point of use instead of vector registers held across a loop.
__constant__ const double kExpCoef[16] = {
    1.4426950408889634, -0x1.62e42fee00000p-1, -0x1.a39ef35793c76p-33,          // 1/ln 2, ln 2 to 32 bits, the rest of ln 2
    1.0 / 6227020800.0, 1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0, 1.0 / 362880.0, 1.0 / 40320.0,
    1.0 / 5040.0, 1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0, 0.5, 1.0};
typedef const __attribute__((address_space(4))) double* ExpCoef;
__device__ __forceinline__ ExpCoef exp_coef() {
    ExpCoef c = (ExpCoef)kExpCoef;
    asm volatile("" : "+s"(c));
    return c;
}
__device__ __forceinline__ double exp_nonpos(double x, ExpCoef c) {
    x = x < -800.0 ? -800.0 : x;                   // the result is 0 from -746 on; NaN stays
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

// The lane id through an opaque instruction: what is derived from it is formed again where it is used
// instead of being held in registers across the zone loop.
__device__ __forceinline__ int opaque_lane() {
    int ln;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
    return ln;
}

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

// Record of an elimination: whether some multiplier exceeded the growth limit or was NaN (a zero, infinite or
// NaN determinant of a 2 x 2 pivot makes one).  One compare each, collected in a scalar mask.
struct TileGuard {
    double limit;
    unsigned long long bad = 0;        // one bit per lane
    __device__ __forceinline__ explicit TileGuard(double l) : limit(l) {}
    __device__ __forceinline__ void see(double x) { bad |= __ballot(!(fabs(x) <= limit)); }
    // by the upper word of the magnitude (abs_key_bits; a NaN's is above any limit's), in the given lanes
    __device__ __forceinline__ void see_key(unsigned key, unsigned long long lanes = ~0ull) {
        bad |= __ballot(key > abs_key_bits(limit)) & lanes;
    }
    // keeps the record current: deferred by the compiler, it would hold every step's multipliers
    __device__ __forceinline__ void pin() { asm volatile("" : "+s"(bad)); }
};

// The sixteen entries of a tile in row order, two per element.
struct TileEntries {
    double2 v[8];
    __device__ __forceinline__ void read(const double* q) {
        const double2* p = reinterpret_cast<const double2*>(q);
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = p[j];
    }
};

// Inverse of a tile in natural order from its entries: every lane solves for its own column with 2 x 2 block
// pivots (two reciprocals in sequence instead of four) and keeps its row.  The pivots are diagonal: no
// exchange between the two halves of the tile.
//
// What the guard watches are the multipliers of the Jacobian's columns, whose dominance bounds them.  The block is
// stored as the transposed Jacobian's (COLS false: the multipliers are those of the stored rows), for the transposed
// solve as the Jacobian's own (COLS true: those of the stored columns).  The multipliers of the Jacobian's rows grow with
// the scattering at no cost in accuracy: watched in the transposed solve, at 100 times the synthetic amplitude they sent
// every system to partial pivoting (4096 systems of 300 zones x 20 groups 9.5 ms, 2.4 so).
template <bool COLS>
__device__ __forceinline__ double tile_inverse(const TileEntries& e, const TileLane& L, TileGuard& G) {
    const double2 r0 = e.v[0], r0b = e.v[1], r1 = e.v[2], r1b = e.v[3], r2 = e.v[4], r2b = e.v[5], r3 = e.v[6],
                  r3b = e.v[7];
    const double d1 = fma(r0.x, r1.y, -(r0.y * r1.x));
    const double i1 = rcp_cubic(d1);
    const double e00 = r1.y * i1, e01 = -(r0.y * i1), e10 = -(r1.x * i1), e11 = r0.x * i1;
    // the multipliers of one half by the other's inverse (those between tiles are seen by the caller); a first
    // determinant that is zero or not finite makes them NaN, a second one makes its reciprocal NaN
    double h00, h01, h10, h11, s00, s01, s10, s11;
    if constexpr (COLS) {                                              // upper half's inverse times the right half
        h00 = fma(e00, r0b.x, e01 * r1b.x), h01 = fma(e00, r0b.y, e01 * r1b.y);
        h10 = fma(e10, r0b.x, e11 * r1b.x), h11 = fma(e10, r0b.y, e11 * r1b.y);
        s00 = fma(-r2.x, h00, fma(-r2.y, h10, r2b.x)), s01 = fma(-r2.x, h01, fma(-r2.y, h11, r2b.y));
        s10 = fma(-r3.x, h00, fma(-r3.y, h10, r3b.x)), s11 = fma(-r3.x, h01, fma(-r3.y, h11, r3b.y));
    } else {                                                           // lower half times the upper's inverse
        h00 = fma(r2.x, e00, r2.y * e10), h01 = fma(r2.x, e01, r2.y * e11);
        h10 = fma(r3.x, e00, r3.y * e10), h11 = fma(r3.x, e01, r3.y * e11);
        s00 = fma(-h00, r0b.x, fma(-h01, r1b.x, r2b.x)), s01 = fma(-h00, r0b.y, fma(-h01, r1b.y, r2b.y));
        s10 = fma(-h10, r0b.x, fma(-h11, r1b.x, r3b.x)), s11 = fma(-h10, r0b.y, fma(-h11, r1b.y, r3b.y));
    }
    const double d2 = fma(s00, s11, -(s01 * s10));
    const double i2 = rcp_cubic(d2);
    G.see(h00);
    G.see(h01);
    G.see(h10);
    G.see(h11);
    G.bad |= __ballot(!(i2 == i2));
    G.pin();
    double x0, x1, x2, x3;
    if constexpr (COLS) {
        const double y0 = fma(e00, L.u0, e01 * L.u1), y1 = fma(e10, L.u0, e11 * L.u1);
        const double t0 = fma(-r2.x, y0, fma(-r2.y, y1, L.u2)), t1 = fma(-r3.x, y0, fma(-r3.y, y1, L.u3));
        x2 = fma(s11, t0, -(s01 * t1)) * i2, x3 = fma(s00, t1, -(s10 * t0)) * i2;
        x0 = fma(-h00, x2, fma(-h01, x3, y0)), x1 = fma(-h10, x2, fma(-h11, x3, y1));
    } else {
        const double t0 = fma(-h00, L.u0, fma(-h01, L.u1, L.u2)), t1 = fma(-h10, L.u0, fma(-h11, L.u1, L.u3));
        x2 = fma(s11, t0, -(s01 * t1)) * i2, x3 = fma(s00, t1, -(s10 * t0)) * i2;
        const double w0 = fma(-r0b.x, x2, fma(-r0b.y, x3, L.u0)), w1 = fma(-r1b.x, x2, fma(-r1b.y, x3, L.u1));
        x0 = fma(e00, w0, e01 * w1), x1 = fma(e10, w0, e11 * w1);
    }
    const double lo = (L.a & 1) ? x1 : x0, hi = (L.a & 1) ? x3 : x2;
    return (L.a & 2) ? hi : lo;
}

// In-place inverse of a block of T x T tiles by block Gauss-Jordan with diagonal tile pivots.  For the
// M-matrices of this method (off-diagonals <= 0, columns or rows dominant) no step subtracts like-signed
// terms except on the diagonal, so entries far below the block's norm keep their relative accuracy.  The coming
// pivot's tile is updated first and gathered through LDS (transposed, so that its inverse comes out as an A
// operand); the rest of a pivot's update runs on the matrix cores under the inversion of the next one.
template <int T, bool COLS>
__device__ __forceinline__ void tile_invert(double (&S)[T][T], const TileLane& L, double* piv, TileGuard& G) {
    double* q = piv + L.g * kPivStride;
    double ct[T], xn = 0.0;
    auto rest = [&](int p) {                                           // all of pivot p's update but the next pivot
#pragma unroll
        for (int ii = 1; ii < T; ++ii) {
            const int i = (p + ii) % T;
#pragma unroll
            for (int jj = 1; jj < T; ++jj) {
                const int j = (p + jj) % T;
                if (ii > 1 || jj > 1 || p == T - 1) S[i][j] = mfma4_neg(ct[i], S[p][j], S[i][j]);
            }
            S[i][p] = mfma4_neg(ct[i], xn, 0.0);
        }
        S[p][p] = xn;
    };
    auto watch = [&](int p) {                                          // minus the multipliers of pivot p's columns
        if constexpr (COLS && T > 1) {
            unsigned m = 0;
#pragma unroll
            for (int i = 0; i < T; ++i)
                if (i != p) m = max(m, abs_key_bits(S[i][p]));
            G.see_key(m);
            G.pin();
        }
    };
    q[4 * L.b + L.a] = S[0][0];
    wave_sync();
#pragma unroll
    for (int p = 0; p < T; ++p) {
        TileEntries e;
        e.read(q);
        wave_sync();
        __builtin_amdgcn_sched_barrier(0);
        if (p > 0) rest(p - 1);
        const double xa = tile_inverse<COLS>(e, L, G);
        if (p > 0) {
#pragma unroll
            for (int j = 0; j < T * (T - 1) - 1; ++j) {                 // one product, then a few vector operations
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (p > 0) watch(p - 1);                                        // its products have come by now
        xn = mfma4(xa, L.id, 0.0);
#pragma unroll
        for (int ii = 1; ii < T; ++ii) ct[(p + ii) % T] = mfma4(S[(p + ii) % T][p], L.id, 0.0);   // A operands of the column
#pragma unroll
        for (int jj = 1; jj < T; ++jj) {
            const int j = (p + jj) % T;
            S[p][j] = mfma4(xa, S[p][j], 0.0);
            if (!COLS) G.see(S[p][j]);
        }
        if (!COLS) G.pin();
        if (p + 1 < T) {
            S[p + 1][p + 1] = mfma4_neg(ct[p + 1], S[p][p + 1], S[p + 1][p + 1]);
            q[4 * L.b + L.a] = S[p + 1][p + 1];
            wave_sync();
        }
    }
    rest(T - 1);
    watch(T - 1);
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

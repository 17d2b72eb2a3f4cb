// FP64 assembly + block elimination + solve of the linearised transport step on 4 x 4 matrix-core tiles
// (diagonal pivots; forward and transposed solves).
//
// Each (species, ray) system is eliminated from both ends of the ray at once: the inward half takes zones
// 0 .. m-1 upwards, the outward half zones I-1 .. m+1 downwards, and both meet in zone m = I/2.  The block
// sequence of a half is that of block-Thomas with the roles of the two off-diagonals taken by "previous" and
// "next" zone, so the arithmetic is the same and the chain of dependent zones half as long.  A wavefront
// holds four blocks of 16 lanes: two systems, both halves of each.
//
// Per step (four zones of a wavefront) the blocks are assembled in registers, reduced by the factor of the
// previous zone still in those registers, and inverted in place (tm_tile.hpp).  The stored block is the
// transpose of the Jacobian's (of the transposed Jacobian's for the adjoint), whose inverse in natural tile
// order is the A operand of the products y = Ahat^-1 g and x = y - C x_next.
//
// What bounds it: with few systems, the chain of zones (540 zones: 2.0 ms, of it 1.2 us per step in the
// back substitution and the rest in assembly and five dependent tile inversions); with the chip full, the
// round trip of C through HBM (119 GB each way at 65536 systems of 540 x 20; 58 ms a launch) together with the issue of
// two waves per SIMD.  The one-row-per-lane kernel before it took 7.7 ms and 122 ms (transposed: 9.0 and
// 130 ms): it exchanged every pivot row through LDS and ran every zone of a ray in sequence.  To fit two
// waves per SIMD at 20 groups, only one matrix is held in registers (the previous factor becomes the Schur
// term in place), the owned cells' state waits in LDS, and what derives from the lane id is formed again
// each step.
#include "tm_kernels.hpp"
#include "tm_tile.hpp"

namespace tmk {

namespace {

__device__ __forceinline__ bool nes_on(const Shape& sh) { return sh.terms & kNes; }

// LDS of a wavefront; VS is the row stride of the group vectors, a multiple of 64 bytes that spreads the
// four blocks over the banks.
template <int T>
struct TileLds {
    static constexpr int NT = 4 * T;
    static constexpr int VS = NT <= 8 ? 8 : (NT <= 24 ? 24 : 40);
    double P[T * T * 16];              // NES shape per tile and lane of a block
    double2 ps[4 * VS];                // psi, coefficient towards the previous zone
    double2 rb[4 * VS];                // right-hand side, coefficient towards the next zone
    double2 ex[4 * VS];                // products of the neighbour factors to the tile's start and end
    double dg[4 * VS];                 // diagonal without the NES sums
    double df[4 * VS];                 // neighbour factors exp(-(eps_{k+1} - eps_k)/T)
    double piv[4 * kPivStride];
    // state of the lane's owned cells at the current zone, used once per step (in LDS to free registers):
    // psi, opacity kappa_a + eta, mean free path, trailing edge's signed area times dH/dpsi of this zone and
    // of the previous one, -(eps_{k+1} - eps_k)
    double own[T > 4 ? 2 : 1][6][64];
};

// Doubles of workspace per wavefront step (four zones): T^2 tiles of 64, then y of the four zones.
template <int T>
constexpr size_t step_doubles() { return (size_t)64 * T * T + 16 * T; }

// The raw values of an owned cell's next zone, as loaded, and the right-hand side of the coming step.
struct NextCell {
    double psi, ka, et, ks, rhs;
};

// Element at a byte offset from a wave-uniform base (scalar base, 32-bit lane offset).
__device__ __forceinline__ double at(const double* base, unsigned off) {
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + off);
}

}  // namespace

namespace {

// Which system, half and zones a lane works on.  Everything but the lane is uniform over the wavefront.
struct Place {
    TileLane L;
    bool half;                         // the half coming from the outer edge
    int delay, dir, I, N;
    double sgn;
    unsigned off0;                     // byte offset of the system's cells from the wavefront's first system
    __device__ __forceinline__ Place(int lane, bool two, unsigned gap, int I_, int N_) : L(lane), I(I_), N(N_) {
        half = L.g & 1;
        delay = half && (I & 1) == 0 ? 1 : 0;                   // the outer half has one zone less
        dir = half ? -1 : 1;
        sgn = half ? -1.0 : 1.0;
        off0 = second(two) ? gap * (unsigned)I * (unsigned)N * 8u : 0u;
    }
    __device__ __forceinline__ bool second(bool two) const { return two && (L.g >> 1); }
    __device__ __forceinline__ int zone_at(int n) const { return half ? I - 1 - (n - delay) : n; }
    __device__ __forceinline__ int clampz(int z) const { return min(max(z, 0), I - 1); }
    __device__ __forceinline__ int clampe(int e) const { return min(max(e, 0), I); }
    // owned group j and its byte offset (clamped to group 0)
    __device__ __forceinline__ int own(int j) const { return 16 * j + 4 * L.b + L.a; }
    __device__ __forceinline__ unsigned own8(int j) const { return own(j) < N ? 8u * own(j) : 0u; }
    __device__ __forceinline__ unsigned cell(int z) const { return off0 + (unsigned)clampz(z) * (unsigned)N * 8u; }
};

}  // namespace

// TRANS: the transposed solve (adjoint).  EXT: lapse and the geometric limiter and boundary compiled in.
template <int T, bool TRANS, bool EXT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(T <= 5 ? 2 : 1)))
void k_factor_tile(FactorArgs A) {
    constexpr int NT = 4 * T;
    constexpr int OWN = T > 4 ? 2 : 1;
    using Lds = TileLds<T>;
    constexpr int VS = Lds::VS;
    __shared__ Lds sm;
    const int lane = threadIdx.x;
    const Shape& sh = A.sh;
    const int N = sh.N, I = sh.I;
    const long long pos0 = (long long)blockIdx.x * 2;
    const bool two = pos0 + 1 < A.nsys;                                 // an odd batch leaves the last wave one system
    const long long first = A.list ? A.list[A.sys0 + pos0] : A.sys0 + pos0;
    const long long other = !two ? first : A.list ? A.list[A.sys0 + pos0 + 1] : first + 1;
    const unsigned gap = (unsigned)(other - first);                     // in systems
    const bool live0 = A.active == nullptr || A.active[first] != 0;
    const bool live1 = two && (A.active == nullptr || A.active[other] != 0);
    if (!live0 && !live1) return;
    {
        const TileLane L(lane);
        for (int t = 0; t < T * T; ++t)                                 // storage row r is k', column q is k
            if (L.g == 0) {
                const int r = 4 * (t / T) + L.a, q = 4 * (t % T) + L.b;
                sm.P[t * 16 + 4 * L.a + L.b] = TRANS ? A.cs->P[r][q] : A.cs->P[q][r];
            }
    }
    wave_sync();

    const int ray0 = (int)(first % sh.R), ray1 = (int)(other % sh.R);
    const int spec0 = (int)(first / sh.R), spec1 = (int)(other / sh.R);
    const size_t base0 = (size_t)first * I * N;
    const double* const psi_b = A.psi + base0;
    const double* const ka_b = A.f.kappa_a + base0;
    const double* const et_b = A.f.eta + base0;
    const double* const ks_b = A.f.kappa_s + base0;
    const double* const rhs_b = A.rhs + base0;
    const double c = sh.c_dt;
    const bool diff = sh.terms & kDiffusion, emabs = sh.terms & kEmAbs, nes = sh.terms & kNes;
    double* ws = reinterpret_cast<double*>(A.wsC) + (size_t)blockIdx.x * 2 * I * NT * (NT + 1);
    const int m = I / 2;                                                // the meeting zone

    NextCell o[OWN];
    double Tz = 1.0, amp = 0.0;
    auto load_next = [&](const Place& P, int z) {                       // raw values of zone z (clamped)
        const unsigned cz = P.cell(z);
#pragma unroll
        for (int j = 0; j < OWN; ++j) {
            o[j].psi = at(psi_b, cz + P.own8(j));
            o[j].ka = at(ka_b, cz + P.own8(j));
            o[j].et = at(et_b, cz + P.own8(j));
            o[j].ks = at(ks_b, cz + P.own8(j));
        }
    };
    auto load_zone = [&](const Place& P, int z) {                       // right-hand side, T and amplitude of zone z
        const unsigned cz = P.cell(z);
#pragma unroll
        for (int j = 0; j < OWN; ++j) o[j].rhs = at(rhs_b, cz + P.own8(j));
        if (nes) {
            Tz = A.f.temp[(size_t)(P.second(two) ? ray1 : ray0) * I + P.clampz(z)];
            amp = A.f.nes_amp[(size_t)(P.second(two) ? other : first) * I + P.clampz(z)];
        }
    };
    auto radius = [&](const Place& P, int e) {
        return A.f.r_edge[(size_t)(P.second(two) ? ray1 : ray0) * (I + 1) + P.clampe(e)];
    };
    // signed area times dH/dpsi_I at the outer boundary, owned group at byte offset k8
    auto outer = [&](const Place& P, unsigned k8, double psi, double lam) -> double {
        if (!diff || sh.outer_bc == 0) return 0.0;
        const int ray = P.second(two) ? ray1 : ray0;
        const double* re = A.f.r_edge + (size_t)ray * (I + 1);
        const double r = re[I];
        double area = r * r;
        if (EXT && A.f.lapse) {
            const double x = A.f.lapse_edge[(size_t)ray * (I + 1) + I];
            area /= x * x;
        }
        if (EXT && sh.outer_bc == 2) {                                   // ghost zone of eq. a62af
            const double rnu = at(A.f.r_nu + (size_t)(P.second(two) ? spec1 : spec0) * N, k8);
            const Ghost gh = outer_ghost(re[I - 1], r, rnu);
            const EdgeFlux e = edge_flux(psi, gh.ratio * psi, lam, gh.D, sh.psi_floor, sh.limiter,
                                         sh.limiter == 2 ? limb_factor(r, rnu) : -1.0);
            return area * (e.dHu + gh.ratio * e.dHv);
        }
        return area;                                                    // free streaming: H = psi of the last zone
    };
    double r_t, r_l, r_b;                                               // edge radii: trailing, leading, next zone's far one
    double iV_prev = 0.0;
    {
        const Place P(lane, two, gap, I, N);
        const int z0 = P.zone_at(0);         // for the outer half the outer zone, or past it when it waits one step
        load_next(P, z0);
#pragma unroll
        for (int j = 0; j < OWN; ++j) {
            const double sig = o[j].ka + o[j].et, lam = rcp_cubic(sig + o[j].ks);
            sm.own[j][0][lane] = o[j].psi;
            sm.own[j][1][lane] = sig;
            sm.own[j][2][lane] = lam;
            sm.own[j][3][lane] = P.half ? outer(P, P.own8(j), o[j].psi, lam) : 0.0;
            sm.own[j][4][lane] = 0.0;
            sm.own[j][5][lane] = (nes && P.own(j) + 1 < N) ? -A.cs->de[P.own(j)] : 0.0;
        }
        load_next(P, z0 + P.dir);
        load_zone(P, z0);
        const int e0 = P.half ? z0 : 1;
        r_t = radius(P, e0 - P.dir);
        r_l = radius(P, e0);
        r_b = radius(P, e0 + P.dir);
    }

    double S[T][T];
    double y[T];
#pragma unroll
    for (int s = 0; s < T; ++s) {
        y[s] = 0.0;
#pragma unroll
        for (int t = 0; t < T; ++t) S[s][t] = 0.0;
    }
    TileGuard guard(A.growth_limit);

    // C and y of step n.  Stored in the middle of the next step, not at the end of their own: loads and stores
    // complete in order, so the wait for the next zone's loads would otherwise include the stores just issued.
    typedef double V2 __attribute__((ext_vector_type(2)));
    auto store = [&](int n, int ln, const TileLane& L) {
        double* q = ws + (size_t)n * step_doubles<T>();
        V2* q2 = reinterpret_cast<V2*>(q) + ln;
#pragma unroll
        for (int j = 0; j < T * T / 2; ++j)
            nt_store(q2 + 64 * j, V2{S[(2 * j) / T][(2 * j) % T], S[(2 * j + 1) / T][(2 * j + 1) % T]});
        if constexpr (T & 1) nt_store(q + 64 * (T * T - 1) + ln, S[T - 1][T - 1]);
        double y1 = 0.0, y2 = 0.0;
        tile_row_to_owner<T>(y, L, y1, y2);
        double* qy = q + 64 * T * T + L.g * NT;
        if (4 * L.b < NT) nt_store(qy + 4 * L.b + L.a, y1);
        if constexpr (T > 4)
            if (16 + 4 * L.b < NT) nt_store(qy + 16 + 4 * L.b + L.a, y2);
    };

    for (int n = 0; n <= m; ++n) {
        const int ln = opaque_lane();
        const Place P(ln, two, gap, I, N);
        const TileLane& L = P.L;
        const bool half = P.half;
        const double sgn = P.sgn;
        const int zc = P.zone_at(n), zn = zc + P.dir;
        const bool idle = n < P.delay;
        const bool lower = TRANS ? L.b > L.a : L.a > L.b;                  // k' > k inside a diagonal tile
        // neighbour factor j of a tile is part of exp(-|eps_k - eps_k'|/T) when min(a,b) <= j < max(a,b)
        const int lo_ab = min(L.a, L.b), hi_ab = max(L.a, L.b);
        const bool has_next = zn >= 0 && zn < I;
        const bool mid = n == m;                                          // uniform
        // ---- geometry of the step
        double iVc = rcp_cubic(sgn * shell_volume(r_t, r_l));
        double iVn = rcp_cubic(sgn * shell_volume(r_l, r_b));
        double sA = sgn * r_l * r_l;
        if (EXT && A.f.lapse) {
            const int ray = P.second(two) ? ray1 : ray0;
            const double* lz = A.f.lapse + (size_t)ray * I;
            const double a0 = lz[P.clampz(zc)], a1 = lz[P.clampz(zn)];
            iVc *= a0 * a0 * a0;
            iVn *= a1 * a1 * a1;
            const double x = A.f.lapse_edge[(size_t)ray * (I + 1) + P.clampe(half ? zc : zc + 1)];
            sA /= x * x;
        }
        const double Dl = fabs(0.5 * (r_l + r_b) - 0.5 * (r_t + r_l));
        iVc = idle ? 0.0 : iVc;
        iVn = has_next ? iVn : 0.0;
        const double cV = c * iVc;
        // ---- owned cells: transport coefficients, right-hand side, neighbour factors
#pragma unroll
        for (int j = 0; j < OWN; ++j) {
            double (&w)[6][64] = sm.own[j];
            const double psi = w[0][ln], sig = w[1][ln], lam = w[2][ln], tc = w[3][ln], to = w[4][ln];
            const bool real = P.own(j) < N;
            const double n_psi = o[j].psi, n_sig = o[j].ka + o[j].et, n_lam = rcp_cubic(n_sig + o[j].ks);
            double ec = 0.0, eo = 0.0;
            if (diff) {
                const double limb = (EXT && sh.limiter == 2)
                                        ? limb_factor(r_l, at(A.f.r_nu + (size_t)(P.second(two) ? spec1 : spec0) * N, P.own8(j))) : -1.0;
                const EdgeFlux e = edge_flux(half ? n_psi : psi, half ? psi : n_psi, sqrt(lam * n_lam), Dl,
                                             sh.psi_floor, sh.limiter, limb);
                ec = sA * (half ? e.dHv : e.dHu);
                eo = sA * (half ? e.dHu : e.dHv);
                if (mid && m + 1 >= I) {                                   // one or two zones: no edge to the next
                    ec = has_next ? ec : (half ? 0.0 : outer(P, P.own8(j), psi, lam));
                    eo = has_next ? eo : 0.0;
                }
            }
            double diag = fma(cV, ec + tc, 1.0);
            if (emabs) diag = fma(c, sig, diag);
            double sch = TRANS ? -c * tc * iV_prev : cV * to;
            double bco = TRANS ? -c * ec * iVn : cV * eo;
            double g = A.rhs_sign * o[j].rhs;
            const bool off = idle || !real;
            diag = off ? 1.0 : diag;
            sch = off ? 0.0 : sch;
            bco = off ? 0.0 : bco;
            g = off ? 0.0 : g;
            w[3][ln] = idle ? tc : -eo;
            w[4][ln] = idle ? to : -ec;
            if (P.own(j) < NT) {
                const int q = L.g * VS + P.own(j);
                sm.ps[q] = make_double2(real ? psi : 0.0, sch);
                sm.rb[q] = make_double2(g, bco);
                sm.dg[q] = diag;
                if (nes) sm.df[q] = P.own(j) + 1 < N ? exp_nonpos(w[5][ln] * rcp_cubic(Tz), exp_coef()) : 0.0;
            }
            w[0][ln] = n_psi;                                            // the next zone becomes the current one
            w[1][ln] = n_sig;
            w[2][ln] = n_lam;
            __builtin_amdgcn_sched_barrier(0);
        }
        wave_sync();
        if (n > 0) store(n - 1, ln, L);
        // ---- loads of the coming step
        const double ampc = idle ? 0.0 : amp;
        {
            const int z1 = P.zone_at(n + 1);
            load_next(P, z1 + P.dir);
            load_zone(P, z1);
        }
        const double r_nb = radius(P, (half ? zc : zc + 1) + 2 * P.dir);

        // ---- Schur update with the previous factor (both neighbours' in the meeting zone)
        if (mid) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const double sc = sm.ps[L.g * VS + 4 * t + L.b].y, bc = sm.rb[L.g * VS + 4 * t + L.b].y;
#pragma unroll
                for (int s = 0; s < T; ++s) S[s][t] = -fma(__shfl_xor(S[s][t], 4), bc, S[s][t] * sc);
            }
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const double sc = -sm.ps[L.g * VS + 4 * t + L.b].y;
#pragma unroll
                for (int s = 0; s < T; ++s) S[s][t] *= sc;
            }
        }
#pragma unroll
        for (int s = 0; s < T; ++s) {                                      // right-hand side, in y's place
            const double sc = sm.ps[L.g * VS + 4 * s + L.a].y;
            const double2 w = sm.rb[L.g * VS + 4 * s + L.a];
            double g = fma(-sc, y[s], w.x);
            if (mid) g = fma(-w.y, __shfl_xor(y[s], 4), g);
            y[s] = g;
        }
        __builtin_amdgcn_sched_barrier(0);
        // ---- NES: -c dt [(1 - psi_k) K^in + psi_k K^out], with M = exp(-|eps_k - eps_k'|/T) as a product of
        //      the factor from the lower group to the start of the next tile, the factors of the tiles
        //      between, and the factor from the start of the upper group's tile
        if (nes) {
            const double* f = sm.df + L.g * VS;
            const double2* ex = sm.ex + L.g * VS;
#pragma unroll
            for (int j = 0; j < OWN; ++j) {
                const int k0 = 16 * j + 4 * L.b;
                if (k0 < NT) {
                    const double f0 = f[k0], f1 = f[k0 + 1], f2 = f[k0 + 2], f3 = f[k0 + 3];
                    const double st = (L.a >= 1 ? f0 : 1.0) * (L.a >= 2 ? f1 : 1.0) * (L.a >= 3 ? f2 : 1.0);
                    const double en = (L.a >= 1 ? 1.0 : f0) * (L.a >= 2 ? 1.0 : f1) * (L.a >= 3 ? 1.0 : f2);
                    sm.ex[L.g * VS + k0 + L.a] = make_double2(st, en * f3);
                }
            }
            wave_sync();
            const double ca = -c * ampc;
            // outer loop over the index of the Jacobian's row tile (k), inner over its column tile (k');
            // in the storage that is (s, t) = (inner, outer), transposed solve (outer, inner)
#pragma unroll
            for (int u = 0; u < T; ++u) {
                const int ko = L.g * VS + 4 * u + (TRANS ? L.a : L.b);
                const double2 xk = sm.ex[ko];
                const double pk = sm.ps[ko].x;
                const double wk = ca * pk, w1 = ca - wk;                    // weights of psi_k and 1 - psi_k
                double acc = 0.0;
                double span = 1.0;                                          // factors of tile u and those between
#pragma unroll
                for (int dv = 0; dv < T; ++dv) {
                    // v = u, u + 1, ..., T - 1, then u - 1, ..., 0
                    const int v = dv < T - u ? u + dv : T - 1 - dv;
                    const int vo = L.g * VS + 4 * v + (TRANS ? L.b : L.a);
                    const int s = TRANS ? u : v, t = TRANS ? v : u;
                    const double Pe = sm.P[(s * T + t) * 16 + 4 * L.a + L.b];
                    const double pv = sm.ps[vo].x;
                    double M;
                    if (v == u) {
                        M = ((lo_ab <= 0 && 0 < hi_ab) ? f[4 * u] : 1.0) * ((lo_ab <= 1 && 1 < hi_ab) ? f[4 * u + 1] : 1.0) *
                            ((lo_ab <= 2 && 2 < hi_ab) ? f[4 * u + 2] : 1.0);
                    } else if (v > u) {
                        span = v == u + 1 ? xk.y : span * ex[4 * v - 4].y;
                        M = span * sm.ex[vo].x;
                    } else {
                        span = v == u - 1 ? xk.x : span * ex[4 * v + 4].y;
                        M = span * sm.ex[vo].y;
                    }
                    const double PM = Pe * M;
                    const bool up = v == u ? lower : v > u;                 // k' > k
                    S[s][t] = fma(up ? w1 : wk, Pe, S[s][t]);
                    S[s][t] = fma(up ? wk : w1, PM, S[s][t]);
                    const double pq = 1.0 - pv;
                    acc = fma(up ? pv : pq, Pe, acc);
                    acc = fma(up ? pq : pv, PM, acc);
                }
                // sum over k': over the rows of the storage, or over its columns for the transposed solve
                if (TRANS) acc = mfma4(mfma4(acc, L.id, 0.0), 1.0, 0.0);
                else acc = mfma4(1.0, acc, 0.0);
                S[u][u] = fma(L.id, c * ampc * acc, S[u][u]);
                wave_sync();                                                // LDS values are read again, not held
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t) S[t][t] = fma(L.id, sm.dg[L.g * VS + 4 * t + L.b], S[t][t]);
        __builtin_amdgcn_sched_barrier(0);

        // ---- Ahat^-1, y = Ahat^-1 g, C = Ahat^-1 diag(b)
        tile_invert<T, TRANS>(S, L, sm.piv, guard);
        double yn[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            double v = 0.0;
#pragma unroll
            for (int s = 0; s < T; ++s) v = mfma4(S[s][t], y[s], v);
            yn[t] = v;
        }
#pragma unroll
        for (int t = 0; t < T; ++t) y[t] = yn[t];
        if (!mid) {
#pragma unroll
            for (int s = 0; s < T; ++s) {
                const double bco = sm.rb[L.g * VS + 4 * s + L.a].y;
#pragma unroll
                for (int t = 0; t < T; ++t) S[s][t] *= bco;
            }
        }
        r_t = r_l;
        r_l = r_b;
        r_b = r_nb;
        iV_prev = iVc;
        wave_sync();
    }

    // ---- growth guard and zero pivots of each system (both halves)
    const Place P(opaque_lane(), two, gap, I, N);
    const TileLane& L = P.L;
    const bool live = (L.g >> 1) ? live1 : live0;
    const long long sys = P.second(two) ? other : first;
    const unsigned long long bad = guard.bad;
    const bool skip = (bad & ((L.g >> 1) ? 0xFF00FF00FF00FF00ull : 0x00FF00FF00FF00FFull)) != 0;
    const bool lead = (lane & 0x37) == 0;                                 // first lane of each system
    if (live && lead && skip) {
        if (A.guard) A.guard[sys] = 1;
        if (A.flags) A.flags[sys] |= 8;
    }
    const bool out = live && !skip;

    // ---- back substitution outwards from the meeting zone, both halves from the inner half's x_m
    double x[T];
#pragma unroll
    for (int s = 0; s < T; ++s) {
        const double met = __shfl_xor(y[s], 4);                            // read with every lane active
        x[s] = P.half ? met : y[s];
    }
    double* const out_b = (A.psi_out ? A.psi_out : A.x) + base0;
    double* const dx_b = A.psi_out && A.dx ? A.dx + base0 : nullptr;
    auto put = [&](int z, bool ok) {
        double x1 = 0.0, x2 = 0.0;
        tile_row_to_owner<T>(x, L, x1, x2);
#pragma unroll
        for (int j = 0; j < OWN; ++j) {
            const double d = j == 0 ? x1 : x2;
            if (ok && P.own(j) < N) {
                const unsigned ci = P.cell(z) + P.own8(j);
                double* p = reinterpret_cast<double*>(reinterpret_cast<char*>(out_b) + ci);
                if (A.psi_out) {
                    *p += d;
                    if (dx_b) *reinterpret_cast<double*>(reinterpret_cast<char*>(dx_b) + ci) = d;
                } else {
                    *p = d;
                }
            }
        }
    };
    double C[T * T], Cn[T * T], yo[2], yon[2];
    auto fetch = [&](int n, double (&c_)[T * T], double (&y_)[2]) {
        const double* q = ws + (size_t)n * step_doubles<T>();
        typedef double V2 __attribute__((ext_vector_type(2)));
        const V2* q2 = reinterpret_cast<const V2*>(q) + lane;
#pragma unroll
        for (int j = 0; j < T * T / 2; ++j) {
            const V2 v = nt_load(q2 + 64 * j);
            c_[2 * j] = v.x;
            c_[2 * j + 1] = v.y;
        }
        if constexpr (T & 1) c_[T * T - 1] = nt_load(q + 64 * (T * T - 1) + lane);
        const double* qy = q + 64 * T * T + L.g * NT;
        y_[0] = 4 * L.b < NT ? nt_load(qy + 4 * L.b + L.a) : 0.0;
        y_[1] = (T > 4 && 16 + 4 * L.b < NT) ? nt_load(qy + 16 + 4 * L.b + L.a) : 0.0;
    };
    if (m > 0) fetch(m - 1, C, yo);
    put(m, out && !P.half);
    for (int n = m - 1; n >= 0; --n) {
        if (n > 0) fetch(n - 1, Cn, yon);
        double xn[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            double v = dpp_quad(t < 4 ? yo[0] : yo[1], t & 3);
#pragma unroll
            for (int s = 0; s < T; ++s) v = mfma4_neg(C[s * T + t], x[s], v);
            xn[t] = v;
        }
#pragma unroll
        for (int t = 0; t < T; ++t) x[t] = xn[t];
        put(P.zone_at(n), out && n >= P.delay);
#pragma unroll
        for (int j = 0; j < T * T; ++j) C[j] = Cn[j];
        yo[0] = yon[0];
        yo[1] = yon[1];
    }
    if (out && lead && A.psi_out) {
        if (A.iters) A.iters[sys] += 1;
        if (A.pending) A.pending[sys] = 1;                                // trial psi + delta awaits the line search
        if (A.alpha) A.alpha[sys] = 1.0;
    }
}

template <int T>
static void launch_tile_t(const FactorArgs& a, bool transpose, hipStream_t st) {
    const dim3 grid((unsigned)((a.nsys + 1) / 2)), block(64);
    const bool ext = a.f.lapse || a.sh.limiter == 2 || a.sh.outer_bc == 2;
    if (transpose) {
        if (ext) hipLaunchKernelGGL((k_factor_tile<T, true, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_factor_tile<T, true, false>), grid, block, 0, st, a);
    } else {
        if (ext) hipLaunchKernelGGL((k_factor_tile<T, false, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_factor_tile<T, false, false>), grid, block, 0, st, a);
    }
}

hipError_t launch_factor_tile(const FactorArgs& a, bool transpose, hipStream_t st) {
    switch (padded_groups(a.sh.N)) {
        case 4: launch_tile_t<1>(a, transpose, st); break;
        case 8: launch_tile_t<2>(a, transpose, st); break;
        case 12: launch_tile_t<3>(a, transpose, st); break;
        case 16: launch_tile_t<4>(a, transpose, st); break;
        case 20: launch_tile_t<5>(a, transpose, st); break;
        case 24: launch_tile_t<6>(a, transpose, st); break;
        case 28: launch_tile_t<7>(a, transpose, st); break;
        case 32: launch_tile_t<8>(a, transpose, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace tmk

// FP64 assembly + block elimination + solve with a wavefront per half ray: the Y_e-coupled blocks,
// and the blocks of one species where there are few systems.
//
// A ray is eliminated from both ends at once by the two wavefronts of a workgroup (zones 0 .. m-1 upwards and
// I-1 .. m+1 downwards, meeting in zone m = I/2).  The transpose of a zone's block is spread over the whole
// wavefront: register S[q][C] of lane 16 a + j holds row 4q + a, column 16C + j.  Each register is a row group
// of four rows by 16 columns, that is, the B operand of v_mfma_f64_4x4x4 with its four blocks taking four
// column groups of the same matrix; the A operand is then a 4 x 4 tile repeated for every block.  Four row groups
// are a result of v_mfma_f64_16x16x4, whose B operand is the same and whose A operand holds 16 rows at once.
//
// Rows and columns of a coupled block: psi of nu_e in 0 .. NT-1, of anti-nu_e in NT .. 2NT-1, Y_e at 2NT (NT =
// N padded to a multiple of 4; padding is identity), in row groups of four: G = 2T + 1.  Per pivot group the
// panel of four columns goes through LDS, every lane inverts the 4 x 4 pivot, and G products per 16 columns
// update the block.  The block is inverted in place, y = Ahat^-1 g and the back substitution are weighted column
// sums over the registers.
//
// One wavefront per half ray, because a 41 x 41 block in one wavefront's registers (33 of them) leaves two
// wavefronts to a SIMD, and the chain of zones is half as long as from one end.  With few rays a step is the
// latency of one wavefront: 11 dependent panels of an LDS round trip, a 4 x 4 inversion (about 75 vector
// operations) and the products.  With many rays the factors' way through memory (13.4 kB a zone, written once and
// read once) comes to half the time.  Per update, 540 zones x 20 groups, residual passes included, against one
// ray per wavefront on 8 x 8 tiles of the vector unit from one end: 90 rays 14.2 -> 3.8 ms, 2048 rays 21.4 -> 14.2 ms,
// 8192 rays 74 -> 54 ms.  Lapse, neutrinosphere options and pairs had partial pivoting
// on the vector unit only; with pairs 90 rays 18 -> 3.8 ms.
// Of a step's 33000 cycles with few rays 17400 are the inversion (630 of each panel's 1585 on the matrix core, which
// does not overlap the vector unit's FP64 work), 9300 the assembly, 4200 the back substitution.
#include "tm_kernels.hpp"
#include "tm_tile.hpp"

namespace tmk {

namespace {

// Sum over the wavefront, in every lane: column sums on the matrix core, then rotations within 16 lanes.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const long long w = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)w, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(w >> 32), CTRL, 0xF, 0xF, true);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double wave_total(double v) {
    v = mfma4(1.0, v, 0.0);
    v = dpp_add<0xB1>(v);              // quad [1,0,3,2]
    v = dpp_add<0x4E>(v);              // quad [2,3,0,1]
    v = dpp_add<0x124>(v);             // row_ror:4
    return dpp_add<0x128>(v);          // row_ror:8
}

// Barrier of the workgroup for what its wavefronts exchange through LDS; memory operations stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int T>
struct CoupledShape {
    static constexpr int NT = 4 * T, NC = 2 * NT, M = NC + 1;
    static constexpr int G = 2 * T + 1, Q = 2 * T, CN = (G + 3) / 4;   // row groups, those of C, column registers
    static constexpr int W = 16 * CN;                                  // columns held
    // column stride of the panel (doubles): 4 past a multiple of 16, so that the 16 lanes that write it (four
    // columns by four rows) hit different banks (a multiple of 16 costs twice the cycles)
    static constexpr int PR = ((4 * G + 11) / 16) * 16 + 4;
    static constexpr int FC = M / 16, REM = M % 16;                    // full column registers, columns past them
};

template <int T, bool EXT>
struct CoupledLds {
    using C = CoupledShape<T>;
    double pan[4 * C::PR];             // pivot panel, column by column
    double psi[C::W], g[C::W], dg[C::W];                         // per row: see the assembly
    double yrow[C::W], ycol[C::W];     // Y_e row and column of the block
    double y[C::W];                    // y of the previous zone; x in the back substitution
    double pe[EXT ? C::W : 1], pm[EXT ? C::W : 1], bz[EXT ? C::NT : 1];   // pair terms
};

// A zone ready for elimination: couplings to the previous and the next zone, right-hand side, and, where a second
// wavefront makes it (AHEAD), the block, lane by lane in the registers' order.
template <int T, bool AHEAD>
struct CoupledZone {
    using C = CoupledShape<T>;
    double sch[C::W], bco[C::W], g[C::W];
    double block[AHEAD ? C::G * C::CN : 1][AHEAD ? 64 : 1];
};

// What a lane owns: row i = lane of the block (species cell i < NC, Y_e at i = NC), and its cell's offset.
template <int T>
struct Owner {
    int species, k;
    bool real;
    size_t cell;
    __device__ __forceinline__ Owner(int lane, const Shape& sh, long long ray) {
        constexpr int NT = 4 * T, NC = 8 * T;
        species = lane < NT ? 0 : 1;
        k = lane - species * NT;
        real = lane < NC && k < sh.N;
        cell = ((size_t)(real ? species : 0) * sh.R + ray) * sh.I * sh.N + (real ? k : 0);
    }
};

}  // namespace

// The wavefront's block: row groups in fours as 16 x 16 results, the last G % 4 on their own.
template <int G, int CN>
struct WaveBlock {
    static constexpr int RF = G / 4, RM = G % 4;
    Vec4 f[RF > 0 ? RF : 1][CN];
    double r[RM > 0 ? RM : 1][CN];
    __device__ __forceinline__ double get(int q, int C) const { return q < 4 * RF ? f[q / 4][C][q % 4] : r[q - 4 * RF][C]; }
    __device__ __forceinline__ void set(int q, int C, double v) {
        if (q < 4 * RF) f[q / 4][C][q % 4] = v;
        else r[q - 4 * RF][C] = v;
    }
};

// In-place inverse of the wavefront's block by block Gauss-Jordan with diagonal tile pivots.  The four columns
// of the pivot's panel go to LDS (and are cleared: the update then leaves minus the panel times the pivot's
// inverse there); every lane reads the pivot tile and its A operands back.  The column register of the coming
// pivot is updated and published first; the rest of a pivot's update runs on the matrix cores under the
// inversion of the next pivot's tile.
template <int G, int CN, int PR, bool COLS = false>
__device__ __forceinline__ void wave_invert(WaveBlock<G, CN>& S, const TileLane& L, int jc, double* pan, TileGuard& guard) {
    constexpr int RF = G / 4, RM = G % 4;
    struct Panel {                                                     // A operands of a pivot's panel
        double f[RF > 0 ? RF : 1], r[RM > 0 ? RM : 1];
    };
    auto publish = [&](int p) {
        if (L.g == (p & 3)) {
#pragma unroll
            for (int q = 0; q < G; ++q) {
                pan[L.b * PR + 4 * q + L.a] = S.get(q, p >> 2);
                S.set(q, p >> 2, 0.0);
            }
        }
        wave_sync();
    };
    auto update = [&](int C, const Panel& l, double u, int p) {
#pragma unroll
        for (int R = 0; R < RF; ++R) S.f[R][C] = mfma16_neg(l.f[R], u, S.f[R][C]);
#pragma unroll
        for (int x = 0; x < RM; ++x)
            if (4 * RF + x != p) S.r[x][C] = mfma4_neg(l.r[x], u, S.r[x][C]);
        S.set(p, C, u);
    };
    auto watch = [&](int p) {                                          // minus the multipliers of panel p's columns
        if constexpr (COLS && G > 1) {
            unsigned m = 0;
#pragma unroll
            for (int q = 0; q < G; ++q)
                if (q != p) m = max(m, abs_key_bits(S.get(q, p >> 2)));
            guard.see_key(m, 0x000F000F000F000Full << (4 * (p & 3)));
            guard.pin();
        }
    };
    auto next_register = [&](int p) { return (p + 1 < G ? p + 1 : p) >> 2; };
    publish(0);
    Panel l_prev{};
    double u_prev[CN] = {};
#pragma unroll
    for (int p = 0; p < G; ++p) {
        const int C0 = p >> 2;
        TileEntries e;                                                 // columns of the pivot: rows of its transpose
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double2* v = reinterpret_cast<const double2*>(pan + j * PR + 4 * p);
            e.v[2 * j] = v[0];
            e.v[2 * j + 1] = v[1];
        }
        Panel l;
#pragma unroll
        for (int R = 0; R < RF; ++R) l.f[R] = pan[L.a * PR + 16 * R + jc];
#pragma unroll
        for (int x = 0; x < RM; ++x) l.r[x] = pan[L.a * PR + 16 * RF + 4 * x + L.b];
        wave_sync();
        __builtin_amdgcn_sched_barrier(0);
        int rest = 0;
        if (p > 0) {                                                   // what is left of the previous update
#pragma unroll
            for (int C = 0; C < CN; ++C)
                if (C != next_register(p - 1)) {
                    update(C, l_prev, u_prev[C], p - 1);
                    rest += RF + RM;
                }
        }
        const double xa = tile_inverse<COLS>(e, L, guard);             // transpose of the inverse: its A operand
#pragma unroll
        for (int j = 0; j < rest; ++j) {                                // one product, then a few vector operations
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        const double xn = mfma4(xa, L.id, 0.0);
        double u[CN];
#pragma unroll
        for (int C = 0; C < CN; ++C) {
            u[C] = mfma4(xa, S.get(p, C), 0.0);                         // zero in the panel's own columns
            if (!COLS) guard.see(u[C]);
        }
        if (!COLS) guard.pin();
        else if (p > 0) watch(p - 1);                                   // while these products are on their way
        u[C0] = L.g == (p & 3) ? xn : u[C0];
        if (C0 < RF) l.f[C0 < RF ? C0 : 0] = L.g == (p & 3) ? 0.0 : l.f[C0 < RF ? C0 : 0];   // the pivot rows stay
        update(next_register(p), l, u[next_register(p)], p);
        if (p + 1 < G) publish(p + 1);
        l_prev = l;
#pragma unroll
        for (int C = 0; C < CN; ++C) u_prev[C] = u[C];
    }
#pragma unroll
    for (int C = 0; C < CN; ++C)
        if (C != next_register(G - 1)) update(C, l_prev, u_prev[C], G - 1);
    watch(G - 1);
}

// EXT: lapse, geometric limiter and boundary, and the pair processes compiled in.  AHEAD: a second wavefront per half
// makes the next zone's block while the first eliminates.
template <int T, bool EXT, bool AHEAD>
__global__ __launch_bounds__(AHEAD ? 256 : 128) __attribute__((amdgpu_waves_per_eu(AHEAD || EXT || T > 5 ? 1 : 2)))
void k_ye_factor_wave(YeFactorArgs A) {
    using X = CoupledShape<T>;
    constexpr int NT = X::NT, NC = X::NC, M = X::M, G = X::G, Q = X::Q, CN = X::CN;
    constexpr int kThreads = AHEAD ? 256 : 128;
    __shared__ CoupledLds<T, EXT> lds[2];
    __shared__ CoupledZone<T, AHEAD> zones[2][AHEAD ? 2 : 1];           // per half: step n in n & 1
    __shared__ double sP[NT * NT];                 // P[k][k'] at [k'][k]
    __shared__ double sG[EXT ? NT * NT : 1];       // pair shape g[k][k'] W_k' / mean W at [k'][k]
    __shared__ double s_eps[NT];
    __shared__ double s_C[Q][CN][64];              // the outer half's last factor, for the meeting zone
    __shared__ double s_y[X::W], s_x[X::W];        // the outer half's y; x of the meeting zone
    __shared__ int s_bad[2];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool half = wave & 1;                                            // the half coming from the outer edge
    const bool second = AHEAD && (wave >> 1);
    const long long ray = A.ray0 + blockIdx.x;
    if (A.active && A.active[ray] == 0) return;                            // all wavefronts
    const Shape& sh = A.sh;
    const int N = sh.N, I = sh.I, R = sh.R;
    const bool diff = sh.terms & kDiffusion, emabs = sh.terms & kEmAbs, nes = sh.terms & kNes;
    const bool pair = EXT && A.y.pair_amp != nullptr;
    for (int j = threadIdx.x; j < NT * NT; j += kThreads) {
        const int kp = j / NT, k = j % NT;
        sP[j] = A.cs->P[k][kp];
        if (EXT) sG[j] = (pair && k < N && kp < N) ? A.y.pair_g[(size_t)k * N + kp] * A.cs->W[kp] / A.cs->wbar : 0.0;
    }
    if (threadIdx.x < NT) s_eps[threadIdx.x] = threadIdx.x < N ? A.cs->eps[threadIdx.x] : 0.0;
    __syncthreads();

    CoupledLds<T, EXT>& sm = lds[half];
    const double c = sh.c_dt;
    const int m = I / 2, delay = half && (I & 1) == 0 ? 1 : 0;         // the outer half has one zone less
    const int dir = half ? -1 : 1;
    const double sgn = half ? -1.0 : 1.0;

    const size_t zb = (size_t)ray * I, eb = (size_t)ray * (I + 1);
    auto clampz = [&](int z) { return min(max(z, 0), I - 1); };
    auto clampe = [&](int e) { return min(max(e, 0), I); };

    double n_psi, n_ka, n_et, n_ks, z_rhs, z_dk, z_de, z_pe = 0.0;      // as loaded: next zone; this zone
    auto load_next = [&](const Owner<T>& O, int z) {
        const size_t ci = O.cell + (size_t)clampz(z) * N;
        n_psi = A.psi[ci];
        n_ka = A.f.kappa_a[ci];
        n_et = A.f.eta[ci];
        n_ks = A.f.kappa_s[ci];
    };
    double Tz = 1.0, amp0 = 0.0, amp1 = 0.0, Y = 0.0, Yn = 0.0, rho = 1.0, gY = 0.0, pamp = 0.0;
    auto load_zone = [&](const Owner<T>& O, int zz) {
        const int z = clampz(zz);
        const size_t ci = O.cell + (size_t)z * N;
        z_rhs = A.G[ci];
        z_dk = z_de = 0.0;
        if (emabs) {
            z_dk = A.y.dka[ci];
            z_de = A.y.deta[ci];
        }
        if (nes || pair) Tz = A.f.temp[zb + z];
        if (nes) {
            amp0 = A.f.nes_amp[zb + z];
            amp1 = A.f.nes_amp[((size_t)R + ray) * I + z];
        }
        Y = A.ye[zb + z];
        Yn = A.y.ye_n[zb + z];
        rho = A.y.rho[zb + z];
        gY = A.GY[zb + z];
        if (pair) {
            pamp = A.y.pair_amp[zb + z];
            z_pe = A.y.pair_eta1[ci];
        }
    };
    // area times dH/dpsi_I at the outer boundary
    auto outer = [&](double rnu, double psi, double lam) -> double {
        if (!diff || sh.outer_bc == 0) return 0.0;
        const double r = A.f.r_edge[eb + I];
        double area = r * r;
        if (EXT && A.f.lapse) {
            const double x = A.f.lapse_edge[eb + I];
            area /= x * x;
        }
        if (EXT && sh.outer_bc == 2) {                                  // ghost zone of eq. a62af
            const Ghost gh = outer_ghost(A.f.r_edge[eb + I - 1], r, rnu);
            const EdgeFlux e = edge_flux(psi, gh.ratio * psi, lam, gh.D, sh.psi_floor, sh.limiter,
                                         sh.limiter == 2 ? limb_factor(r, rnu) : -1.0);
            return area * (e.dHu + gh.ratio * e.dHv);
        }
        return area;                                                   // free streaming: H = psi of the last zone
    };
    auto radius_nu = [&](const Owner<T>& O) {
        return EXT && A.f.r_nu && O.real ? A.f.r_nu[(size_t)O.species * N + O.k] : 1.0;
    };
    const int z0 = half ? I - 1 : 0;
    double psi, sig, lam, tc, to = 0.0;                                 // this zone; trailing edge
    double r_t = 0.0, r_l = 0.0, r_b = 0.0;
    if (!AHEAD || second) {
        const Owner<T> O(lane, sh, ray);
        load_next(O, z0);
        psi = n_psi;
        sig = n_ka + n_et;
        lam = rcp_cubic(sig + n_ks);
        tc = half ? outer(radius_nu(O), psi, lam) : 0.0;
        load_next(O, z0 + dir);
        load_zone(O, z0);
        const int e0 = half ? I - 1 : 1;
        r_t = A.f.r_edge[clampe(e0 - dir) + eb];
        r_l = A.f.r_edge[clampe(e0) + eb];
        r_b = A.f.r_edge[clampe(e0 + dir) + eb];
    }

    WaveBlock<G, CN> S;
#pragma unroll
    for (int q = 0; q < G; ++q)
#pragma unroll
        for (int C = 0; C < CN; ++C) S.set(q, C, 0.0);
    if (!second && lane < X::W) {
        sm.y[lane] = 0.0;
        sm.yrow[lane] = sm.ycol[lane] = sm.psi[lane] = sm.g[lane] = 0.0;
        sm.dg[lane] = 1.0;
        for (int b = 0; b < (AHEAD ? 2 : 1); ++b)
            zones[half][b].sch[lane] = zones[half][b].bco[lane] = zones[half][b].g[lane] = 0.0;
    }
    __syncthreads();
    TileGuard guard(A.growth_limit);
    const size_t SZ = (size_t)M * M + 1;                               // slot of a zone (M is odd)
    double* ws = A.ws + (size_t)blockIdx.x * I * SZ;
    typedef double V2 __attribute__((ext_vector_type(2)));

    // C and y of the zone of step n
    auto store = [&](int n, int ln) {
        const int jc = ln & 15, a = ln >> 4;
        double* slot = ws + (size_t)(half ? I - 1 - (n - delay) : n) * SZ;
#pragma unroll
        for (int C = 0; C < X::FC; ++C)
#pragma unroll
            for (int q = 0; q < Q; q += 2)
                nt_store(reinterpret_cast<V2*>(slot) + (C * T + q / 2) * 64 + ln, V2{S.get(q, C), S.get(q + 1, C)});
        if (X::REM && jc < X::REM) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
                nt_store(slot + 64 * Q * X::FC + 4 * X::REM * q + X::REM * a + jc, S.get(q, X::FC < CN ? X::FC : 0));
        }
        if (ln < M) nt_store(slot + (size_t)NC * M + ln, sm.y[ln]);
    };


    // Owned rows of the zone of step n: transport coefficients, Y_e terms, right-hand side; then loads of what comes
    double iT = 1.0, a0 = 0.0, a1 = 0.0, pa = 0.0;
    auto own = [&](int n, CoupledZone<T, AHEAD>& out) {
        // what derives from the lane id is formed again each step instead of being held across it
        const int ln = opaque_lane();
        const Owner<T> O(ln, sh, ray);
        const bool real = O.real;
        const double rnu = radius_nu(O);
        const double qs = O.species == 0 ? 1.0 : -1.0;                 // nu_e carries +1, anti-nu_e -1
        const double Wk = real ? A.cs->W[O.k] : 0.0;
        const int zc = half ? I - 1 - (n - delay) : n, zn = zc + dir;
        const bool has_next = zn >= 0 && zn < I;
        const ExpCoef coef = exp_coef();
        // ---- owned rows: transport coefficients, Y_e terms, right-hand side
        double alz = 1.0, iVc = rcp_cubic(sgn * shell_volume(r_t, r_l)), sA = sgn * r_l * r_l;
        if (EXT && A.f.lapse) {
            alz = A.f.lapse[zb + zc];
            iVc *= alz * alz * alz;
            const double x = A.f.lapse_edge[eb + clampe(half ? zc : zc + 1)];
            sA /= x * x;
        }
        const double cV = c * iVc;
        const double n_sig = n_ka + n_et, n_lam = rcp_cubic(n_sig + n_ks);
        double ec = 0.0, eo = 0.0;
        if (diff) {
            if (has_next) {
                const double Dl = fabs(0.5 * (r_l + r_b) - 0.5 * (r_t + r_l));
                const double limb = (EXT && sh.limiter == 2) ? limb_factor(r_l, rnu) : -1.0;
                const EdgeFlux e = edge_flux(half ? n_psi : psi, half ? psi : n_psi, sqrt(lam * n_lam), Dl, sh.psi_floor,
                                             sh.limiter, limb);
                ec = sA * (half ? e.dHv : e.dHu);
                eo = sA * (half ? e.dHu : e.dHv);
            } else if (!half) {
                ec = outer(rnu, psi, lam);
            }
        }
        const double dy = Y - Yn, dk = alz * z_dk, de = alz * z_de;
        const double zt = kFourPiOverHc3 * kBaryonMassG / (rho * alz * alz * alz);
        double diag = fma(cV, ec + tc, 1.0), yrow = 0.0, ycol = 0.0, ysum = 0.0;
        if (emabs) {
            diag += c * sig + c * dy * (dk + de);
            ycol = c * (dk * psi - de * (1.0 - psi));
            yrow = -qs * c * zt * Wk * (sig + dy * (dk + de));
            ysum = real ? qs * Wk * (de * (1.0 - psi) - dk * psi) : 0.0;
            ysum = wave_total(ysum);
        }
        if (ln <= NC) {
            out.sch[ln] = real ? cV * to : 0.0;
            out.bco[ln] = real ? cV * eo : 0.0;
            out.g[ln] = real ? A.rhs_sign * z_rhs : (ln == NC ? A.rhs_sign * gY : 0.0);
            sm.psi[ln] = real ? psi : 0.0;
            sm.dg[ln] = real ? diag : (ln == NC && emabs ? fma(c * zt, ysum, 1.0) : 1.0);
            sm.yrow[ln] = real ? yrow : 0.0;
            sm.ycol[ln] = real ? ycol : 0.0;
            if (EXT && pair) {
                const double Rz = 0.5 * (A.f.r_edge[eb + zc] + A.f.r_edge[eb + zc + 1]);
                sm.pe[ln] = real ? z_pe : 0.0;
                sm.pm[ln] = real ? pair_limb_cosine(rnu / Rz) : 0.0;
                if (ln < NT) sm.bz[ln] = real ? exp_nonpos(-s_eps[ln] * rcp_cubic(Tz), coef) : 0.0;
            }
        }
        tc = -eo;                                                      // the next zone becomes the current one
        to = -ec;
        psi = n_psi;
        sig = n_sig;
        lam = n_lam;
        wave_sync();
        iT = rcp_cubic(Tz);
        a0 = amp0;
        a1 = amp1;
        pa = pamp;
        load_next(O, zn + dir);
        load_zone(O, zn);
        r_t = r_l;
        r_l = r_b;
        r_b = A.f.r_edge[eb + clampe((half ? zc : zc + 1) + 2 * dir)];
        __builtin_amdgcn_sched_barrier(0);
    };
    // Column register C of the zone's block before elimination, rows 4q + a: scattering and pair terms per column k of
    // the stored transpose and row k' = 4u + a, the Y_e column and row, and the diagonal
    auto column = [&](int C, int ln, double (&B)[G]) {
            const int jc = ln & 15;
            const TileLane L(ln);
            const ExpCoef coef = exp_coef();
#pragma unroll
            for (int q = 0; q < G; ++q) B[q] = 0.0;
            const bool has0 = 4 * C < T, has1 = 4 * C + 3 >= T && 4 * C < 2 * T;   // compile-time
            const int cg = 4 * C + L.g;                                 // column group: species, tile
            const int sc = cg < T ? 0 : 1, tt = cg - sc * T;
            const bool in = cg < 2 * T;
            const int k = in ? 4 * tt + L.b : 0;
            const double m0 = cg < T ? 1.0 : 0.0, m1 = (cg >= T && in) ? 1.0 : 0.0;
            double dgv = sm.dg[16 * C + jc];
            const double pk = sm.psi[16 * C + jc];
            if (nes && (has0 || has1)) {
                const double camp = in ? c * (sc ? a1 : a0) : 0.0;
                const double wk = -camp * pk, w1 = -camp - wk;          // weights of psi_k and 1 - psi_k
                const double ek = s_eps[k];
                double acc = 0.0;
#pragma unroll
                for (int u = 0; u < T; ++u) {
                    const int kp = 4 * u + L.a;
                    const double P = sP[kp * NT + k];
                    const double PM = P * exp_nonpos(-fabs(s_eps[kp] - ek) * iT, coef);
                    const double pv = sm.psi[(sc ? NT : 0) + kp];
                    const bool up = kp > k;
                    const double e = fma(up ? wk : w1, PM, (up ? w1 : wk) * P);
                    if (has0) B[u] = fma(m0, e, B[u]);
                    if (has1) B[T + u] = fma(m1, e, B[T + u]);
                    const double pq = 1.0 - pv;
                    acc = fma(up ? pv : pq, P, acc);
                    acc = fma(up ? pq : pv, PM, acc);
                }
                dgv = fma(camp, mfma4(1.0, acc, 0.0), dgv);
            }
            if (EXT && pair && (has0 || has1)) {
                const int self = in ? 16 * C + jc : 0;
                const double bk = sm.bz[k], ek = sm.pe[self], mk = sm.pm[self];
                const double w = in ? pa : 0.0;
                double acc = 0.0;
#pragma unroll
                for (int u = 0; u < T; ++u) {
                    const int kp = 4 * u + L.a, o = (sc ? 0 : NT) + kp;
                    const double qa = w * sG[kp * NT + k];
                    const double qp = qa * bk * sm.bz[kp];
                    const double qx = qa * pair_chi(ek, sm.pe[o], mk, sm.pm[o]);
                    const double pv = sm.psi[o];
                    const double e = c * fma(1.0 - pk, qp, pk * qx);
                    if (has0) B[T + u] = fma(m0, e, B[T + u]);
                    if (has1) B[u] = fma(m1, e, B[u]);
                    acc += fma(qp, 1.0 - pv, qx * pv);
                }
                dgv = fma(c, mfma4(1.0, acc, 0.0), dgv);
            }
            if (emabs) {
                B[2 * T] = fma(L.a == 0 ? 1.0 : 0.0, sm.ycol[16 * C + jc], B[2 * T]);
                if (C == (2 * T) >> 2) {
                    const double isY = (L.g == ((2 * T) & 3) && L.b == 0) ? 1.0 : 0.0;
#pragma unroll
                    for (int q = 0; q < Q; ++q) B[q] = fma(isY, sm.yrow[4 * q + L.a], B[q]);
                }
            }
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (4 * C + x < G) {
                    const double on = (L.g == x && L.a == L.b) ? 1.0 : 0.0;
                    B[4 * C + x] = fma(on, dgv, B[4 * C + x]);
                }
    };
    auto assemble = [&](int n) {
        CoupledZone<T, AHEAD>& out = zones[half][AHEAD ? n & 1 : 0];
        own(n, out);
        const int ln = opaque_lane();
#pragma unroll
        for (int C = 0; C < CN; ++C) {
            double B[G];
            column(C, ln, B);
#pragma unroll
            for (int q = 0; q < G; ++q) out.block[AHEAD ? C * G + q : 0][AHEAD ? ln : 0] = B[q];
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    if (AHEAD) {
        if (second && delay == 0 && (m > 0 || !half)) assemble(0);
        lds_barrier();
    }
    for (int n = 0; n <= m; ++n) {
        const bool mid = n == m;
        if (mid) {                                                     // the outer half hands its last factor over
            if (half && !second) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int C = 0; C < CN; ++C) s_C[q][C][lane] = S.get(q, C);
                if (lane < X::W) s_y[lane] = sm.y[lane];
                const bool bad = guard.bad != 0ull;
                if (lane == 0) s_bad[1] = bad;
            }
            if (AHEAD) lds_barrier();
            else __syncthreads();
        }
        if (second) {
            if (n + 1 >= delay && n + 1 < m + (half ? 0 : 1)) assemble(n + 1);
        } else if (n >= delay && !(mid && half)) {
            CoupledZone<T, AHEAD>& in = zones[half][AHEAD ? n & 1 : 0];
            if (!AHEAD) own(n, in);
            const int ln = opaque_lane(), jc = ln & 15;
            const TileLane L(ln);
            if (ln <= NC) {
                double g = fma(-in.sch[ln], sm.y[ln], in.g[ln]);
                if (mid) g = fma(-in.bco[ln], s_y[ln], g);
                sm.g[ln] = g;
            }
            // ---- the block, with the Schur term of the previous factor (both neighbours' in the meeting zone)
#pragma unroll
            for (int C = 0; C < CN; ++C) {
                double B[G];
                if constexpr (!AHEAD) column(C, ln, B);
                const double sc = -in.sch[16 * C + jc], bc = in.bco[16 * C + jc];
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    S.set(q, C, fma(S.get(q, C), sc, AHEAD ? in.block[AHEAD ? C * G + q : 0][AHEAD ? ln : 0] : B[q]));
                    if (mid && q < Q) S.set(q, C, fma(-s_C[q][C][ln], bc, S.get(q, C)));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // ---- Ahat^-1, y = Ahat^-1 g, C = Ahat^-1 diag(b)
            wave_invert<G, CN, X::PR>(S, L, jc, sm.pan, guard);
            double yc[CN];
#pragma unroll
            for (int C = 0; C < CN; ++C) yc[C] = 0.0;
#pragma unroll
            for (int q = 0; q < G; ++q) {
                const double g = sm.g[4 * q + L.a];
#pragma unroll
                for (int C = 0; C < CN; ++C) yc[C] = fma(S.get(q, C), g, yc[C]);
            }
#pragma unroll
            for (int C = 0; C < CN; ++C) yc[C] = mfma4(1.0, yc[C], 0.0);
            if (L.a == 0) {
#pragma unroll
                for (int C = 0; C < CN; ++C) sm.y[16 * C + jc] = yc[C];
            }
            wave_sync();
            if (!mid) {
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    const double b = q < Q ? in.bco[4 * q + L.a] : 0.0;     // Y_e has no neighbours
#pragma unroll
                    for (int C = 0; C < CN; ++C) S.set(q, C, S.get(q, C) * b);
                }
                store(n, ln);
            }
        }
        if (AHEAD && !mid) lds_barrier();
    }
    if (wave == 0) {
        const bool bad = guard.bad != 0ull;
        if (lane == 0) s_bad[0] = bad;
        if (lane < X::W) s_x[lane] = sm.y[lane];
    }
    __syncthreads();
    // a ray whose growth guard tripped is left untouched and marked for the partial-pivoting re-run
    const bool bad = s_bad[0] || s_bad[1];
    if (A.redo && threadIdx.x == 0) A.redo[ray] = bad ? 1 : 0;
    if (bad || second) return;

    // ---- back substitution outwards from the meeting zone
    const int lb = opaque_lane(), jc = lb & 15;                         // jc: column within a register
    const TileLane L(lb);
    const Owner<T> O(lb, sh, ray);
    auto put = [&](int z, double d) {
        if (O.real) {
            const size_t ci = O.cell + (size_t)z * N;
            A.psi_out[ci] += d;
            A.dx[ci] = d;
        } else if (lane == NC) {
            A.ye_out[zb + z] += d;
            A.dY[zb + z] = d;
        }
    };
    if (lane < X::W) sm.y[lane] = s_x[lane];
    if (!half) put(m, lane < X::W ? s_x[lane] : 0.0);
    wave_sync();
    double Cb[2][Q][CN], yb[2][CN];                                     // y in column form
    auto fetch = [&](int n, double (&c_)[Q][CN], double (&y_)[CN]) {
        const int z = half ? I - 1 - (n - delay) : n;
        const double* slot = ws + (size_t)z * SZ;
#pragma unroll
        for (int C = 0; C < X::FC; ++C)
#pragma unroll
            for (int q = 0; q < Q; q += 2) {
                const V2 v = nt_load(reinterpret_cast<const V2*>(slot) + (C * T + q / 2) * 64 + lane);
                c_[q][C] = v.x;
                c_[q + 1][C] = v.y;
            }
        if constexpr (X::REM > 0) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
                c_[q][X::FC] = jc < X::REM ? nt_load(slot + 64 * Q * X::FC + 4 * X::REM * q + X::REM * L.a + jc) : 0.0;
        }
#pragma unroll
        for (int C = 0; C < CN; ++C) y_[C] = 16 * C + jc < M ? nt_load(slot + (size_t)NC * M + 16 * C + jc) : 0.0;
    };
    auto step = [&](int n, const double (&c_)[Q][CN], const double (&y_)[CN]) {
        double acc[CN];
#pragma unroll
        for (int C = 0; C < CN; ++C) acc[C] = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const double x = sm.y[4 * q + L.a];
#pragma unroll
            for (int C = 0; C < (X::REM ? X::FC + 1 : X::FC); ++C) acc[C] = fma(c_[q][C], x, acc[C]);
        }
#pragma unroll
        for (int C = 0; C < CN; ++C) acc[C] = y_[C] - mfma4(1.0, acc[C], 0.0);
        wave_sync();
        if (L.a == 0) {
#pragma unroll
            for (int C = 0; C < CN; ++C) sm.y[16 * C + jc] = acc[C];
        }
        wave_sync();
        const double x = lane < X::W ? sm.y[lane] : 0.0;                 // owner form
        put(half ? I - 1 - (n - delay) : n, x);
    };
    int n = m - 1;
    if (n >= delay) fetch(n, Cb[0], yb[0]);
    for (; n >= delay; n -= 2) {
        if (n - 1 >= delay) fetch(n - 1, Cb[1], yb[1]);
        step(n, Cb[0], yb[0]);
        if (n - 1 < delay) break;
        if (n - 2 >= delay) fetch(n - 2, Cb[0], yb[0]);
        step(n - 1, Cb[1], yb[1]);
    }
    if (threadIdx.x == 0) {
        A.iters[ray] += 1;
        A.pending[ray] = 1;                                            // trial psi + delta awaits the line search
        A.alpha[ray] = 1.0;
    }
}

// Up to this many rays, one workgroup to each CU (the two zones handed over per half fill most of its LDS), a second
// wavefront per half assembles the blocks of the general form, whose pair terms are as long as a third of the
// elimination: 90 rays 5.1 -> 4.1 ms an update, 256 rays 5.3 -> 4.3, 512 rays 5.9 -> 8.1.  The plain form gains
// nothing (3.95 against 3.98 ms at 90 rays): what its own assembly takes, the elimination gives back in registers.
constexpr long long kAheadRays = 256;

template <int T>
static void launch_wave_t(const YeFactorArgs& a, bool ext, hipStream_t st) {
    const dim3 grid((unsigned)a.nray);
    if (!ext) {
        hipLaunchKernelGGL((k_ye_factor_wave<T, false, false>), grid, dim3(128), 0, st, a);
        return;
    }
    if constexpr (T <= 6) {                            // two zones ahead per half: 160 KB of LDS at 24 groups
        if (a.sh.R <= kAheadRays) {
            hipLaunchKernelGGL((k_ye_factor_wave<T, true, true>), grid, dim3(256), 0, st, a);
            return;
        }
    }
    hipLaunchKernelGGL((k_ye_factor_wave<T, true, false>), grid, dim3(128), 0, st, a);
}

hipError_t launch_ye_factor_wave(const YeFactorArgs& a, hipStream_t st) {
    if (!a.redo) return hipErrorInvalidValue;
    const bool ext = a.sh.limiter == 2 || a.sh.outer_bc == 2 || a.y.pair_amp || a.f.lapse;
    switch (padded_groups(a.sh.N)) {
        case 4: launch_wave_t<1>(a, ext, st); break;
        case 8: launch_wave_t<2>(a, ext, st); break;
        case 12: launch_wave_t<3>(a, ext, st); break;
        case 16: launch_wave_t<4>(a, ext, st); break;
        case 20: launch_wave_t<5>(a, ext, st); break;
        case 24: launch_wave_t<6>(a, ext, st); break;
        case 28: launch_wave_t<7>(a, ext, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- single species, few systems
//
// The same layout for an N x N block, and two wavefronts to a half: few systems leave the chip idle, so the time of
// a step is that of its dependent operations.  Of these only the Schur term, the inversion and y depend on the zone
// before; the rest of the block (transport coefficients, one exponential per entry, the diagonal) is made by the
// half's second wavefront, on another SIMD, one zone ahead, and handed over in LDS with one barrier a step.
// 540 zones x 20 groups, 24 systems: 2.00 ms on tiles, 1.45 with one wavefront to a half, 1.00 here; 512 systems
// 2.00, 1.99, 1.35.
namespace {

template <int T>
struct SingleShape {
    static constexpr int NT = 4 * T, CN = (T + 3) / 4, W = 16 * CN;
    static constexpr int PR = ((4 * T + 11) / 16) * 16 + 4;
    static constexpr int FC = NT / 16, REM = NT % 16;
};

// A zone as its half's second wavefront hands it to the first: the block before elimination (lane by lane, in the
// registers' order), the couplings to the previous and the next zone and the right-hand side.
template <int T>
struct ZoneBlock {
    using C = SingleShape<T>;
    double block[T * C::CN][64];
    double sch[C::W], bco[C::W], g[C::W];
};

template <int T>
struct SingleLds {
    using C = SingleShape<T>;
    ZoneBlock<T> zone[2];              // of step n in n & 1
    double pan[4 * C::PR];
    double psi[C::W], dg[C::W], g[C::W];
    double y[C::W];                    // y of the previous zone; x in the back substitution
};

}  // namespace

// One (species, ray) system per workgroup, TRANS the transposed solve, EXT the lapse and the geometric options.
template <int T, bool TRANS, bool EXT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_factor_wave(FactorArgs A) {
    using X = SingleShape<T>;
    constexpr int NT = X::NT, CN = X::CN;
    __shared__ SingleLds<T> lds[2];
    __shared__ double sP[NT * X::W];               // P[k][k'] with k the column: [row][column], zero beyond NT
    __shared__ double sPt[TRANS ? NT * X::W : 1];  // P[row][column]
    __shared__ double s_eps[X::W];
    __shared__ double s_C[T][CN][64];              // the outer half's last factor, for the meeting zone
    __shared__ double s_y[X::W], s_x[X::W];        // the outer half's y; x of the meeting zone
    __shared__ int s_bad[2];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool half = wave & 1;                                            // the half coming from the outer edge
    const bool assembles = wave >> 1;                                      // the half's second wavefront
    const long long sys = A.list ? A.list[A.sys0 + blockIdx.x] : A.sys0 + blockIdx.x;
    if (A.active && A.active[sys] == 0) return;                            // all wavefronts
    const Shape& sh = A.sh;
    const int N = sh.N, I = sh.I;
    const bool diff = sh.terms & kDiffusion, emabs = sh.terms & kEmAbs, nes = sh.terms & kNes;
    for (int j = threadIdx.x; j < NT * X::W; j += 256) {
        const int r = j / X::W, q = j % X::W;
        sP[j] = q < NT ? A.cs->P[q][r] : 0.0;
        if (TRANS) sPt[j] = q < NT ? A.cs->P[r][q] : 0.0;
    }
    if (threadIdx.x < X::W) s_eps[threadIdx.x] = threadIdx.x < N ? A.cs->eps[threadIdx.x] : 0.0;
    __syncthreads();

    SingleLds<T>& sm = lds[half];
    const double c = sh.c_dt;
    const int m = I / 2, delay = half && (I & 1) == 0 ? 1 : 0;         // the outer half has one zone less
    const int dir = half ? -1 : 1;
    const double sgn = half ? -1.0 : 1.0;
    const int ray = (int)(sys % sh.R), spec = (int)(sys / sh.R);
    const size_t cb = (size_t)sys * I * N, zb = (size_t)ray * I, eb = (size_t)ray * (I + 1);
    auto clampz = [&](int z) { return min(max(z, 0), I - 1); };
    auto clampe = [&](int e) { return min(max(e, 0), I); };
    auto group = [&](int ln) { return ln < N ? ln : 0; };              // owner lane i owns group i

    double n_psi, n_ka, n_et, n_ks, z_rhs;                              // as loaded: next zone; this zone
    auto load_next = [&](int k, int z) {
        const size_t ci = cb + (size_t)clampz(z) * N + k;
        n_psi = A.psi[ci];
        n_ka = A.f.kappa_a[ci];
        n_et = A.f.eta[ci];
        n_ks = A.f.kappa_s[ci];
    };
    double Tz = 1.0, amp = 0.0;
    auto load_zone = [&](int k, int zz) {
        const int z = clampz(zz);
        z_rhs = A.rhs[cb + (size_t)z * N + k];
        if (nes) {
            Tz = A.f.temp[zb + z];
            amp = A.f.nes_amp[(size_t)sys * I + z];
        }
    };
    // area times dH/dpsi_I at the outer boundary
    auto outer = [&](double rnu, double psi, double lam) -> double {
        if (!diff || sh.outer_bc == 0) return 0.0;
        const double r = A.f.r_edge[eb + I];
        double area = r * r;
        if (EXT && A.f.lapse) {
            const double x = A.f.lapse_edge[eb + I];
            area /= x * x;
        }
        if (EXT && sh.outer_bc == 2) {                                  // ghost zone of eq. a62af
            const Ghost gh = outer_ghost(A.f.r_edge[eb + I - 1], r, rnu);
            const EdgeFlux e = edge_flux(psi, gh.ratio * psi, lam, gh.D, sh.psi_floor, sh.limiter,
                                         sh.limiter == 2 ? limb_factor(r, rnu) : -1.0);
            return area * (e.dHu + gh.ratio * e.dHv);
        }
        return area;                                                   // free streaming: H = psi of the last zone
    };
    auto radius_nu = [&](int k) { return EXT && A.f.r_nu ? A.f.r_nu[(size_t)spec * N + k] : 1.0; };
    const int z0 = half ? I - 1 : 0;
    double psi, sig, lam, tc, to = 0.0, iV_prev = 0.0;                  // this zone; trailing edge
    double r_t = 0.0, r_l = 0.0, r_b = 0.0;
    if (assembles) {
        const int k = group(lane);
        load_next(k, z0);
        psi = n_psi;
        sig = n_ka + n_et;
        lam = rcp_cubic(sig + n_ks);
        tc = half ? outer(radius_nu(k), psi, lam) : 0.0;
        load_next(k, z0 + dir);
        load_zone(k, z0);
        const int e0 = half ? I - 1 : 1;
        r_t = A.f.r_edge[clampe(e0 - dir) + eb];
        r_l = A.f.r_edge[clampe(e0) + eb];
        r_b = A.f.r_edge[clampe(e0 + dir) + eb];
    }


    WaveBlock<T, CN> S;
#pragma unroll
    for (int q = 0; q < T; ++q)
#pragma unroll
        for (int C = 0; C < CN; ++C) S.set(q, C, 0.0);
    if (!assembles && lane < X::W) {
        sm.psi[lane] = sm.g[lane] = sm.y[lane] = 0.0;
        sm.dg[lane] = 1.0;
        for (int b = 0; b < 2; ++b) sm.zone[b].sch[lane] = sm.zone[b].bco[lane] = sm.zone[b].g[lane] = 0.0;
    }
    __syncthreads();
    TileGuard guard(A.growth_limit);
    constexpr size_t SZ = (size_t)NT * (NT + 1);                       // slot of a zone
    double* ws = reinterpret_cast<double*>(A.wsC) + (size_t)blockIdx.x * I * SZ;
    typedef double V2 __attribute__((ext_vector_type(2)));

    // C and y of the zone of step n
    auto store = [&](int n, int ln) {
        const int jc = ln & 15, a = ln >> 4;
        double* slot = ws + (size_t)(half ? I - 1 - (n - delay) : n) * SZ;
#pragma unroll
        for (int C = 0; C < X::FC; ++C) {
#pragma unroll
            for (int q = 0; q + 1 < T; q += 2)
                nt_store(reinterpret_cast<V2*>(slot + 64 * T * C) + 32 * q + ln, V2{S.get(q, C), S.get(q + 1, C)});
            if (T & 1) nt_store(slot + 64 * T * C + 64 * (T - 1) + ln, S.get(T - 1, C));
        }
        if (X::REM && jc < X::REM) {
#pragma unroll
            for (int q = 0; q < T; ++q)
                nt_store(slot + 64 * T * X::FC + 4 * X::REM * q + X::REM * a + jc, S.get(q, X::FC < CN ? X::FC : 0));
        }
        if (ln < NT) nt_store(slot + (size_t)NT * NT + ln, sm.y[ln]);
    };


    // Zone of step n into its place: transport coefficients and right-hand side of the owned groups, then scattering
    // terms and diagonal, per column of the stored matrix and row 4u + a
    auto assemble = [&](int n) {
        ZoneBlock<T>& out = sm.zone[n & 1];
        // what derives from the lane id is formed again each step instead of being held across it
        const int ln = opaque_lane(), jc = ln & 15, k = group(ln);
        const TileLane L(ln);
        const bool real = ln < N;
        const int zc = half ? I - 1 - (n - delay) : n, zn = zc + dir;
        const bool has_next = zn >= 0 && zn < I;
        const ExpCoef coef = exp_coef();
        // ---- owned groups: transport coefficients, right-hand side
        double iVc = rcp_cubic(sgn * shell_volume(r_t, r_l)), iVn = 0.0, sA = sgn * r_l * r_l;
        if (TRANS && has_next) iVn = rcp_cubic(sgn * shell_volume(r_l, r_b));
        if (EXT && A.f.lapse) {
            const double a0 = A.f.lapse[zb + zc], a1 = A.f.lapse[zb + clampz(zn)];
            iVc *= a0 * a0 * a0;
            iVn *= a1 * a1 * a1;
            const double x = A.f.lapse_edge[eb + clampe(half ? zc : zc + 1)];
            sA /= x * x;
        }
        const double cV = c * iVc;
        const double n_sig = n_ka + n_et, n_lam = rcp_cubic(n_sig + n_ks);
        double ec = 0.0, eo = 0.0;
        if (diff) {
            if (has_next) {
                const double Dl = fabs(0.5 * (r_l + r_b) - 0.5 * (r_t + r_l));
                const double limb = (EXT && sh.limiter == 2) ? limb_factor(r_l, radius_nu(k)) : -1.0;
                const EdgeFlux e = edge_flux(half ? n_psi : psi, half ? psi : n_psi, sqrt(lam * n_lam), Dl, sh.psi_floor,
                                             sh.limiter, limb);
                ec = sA * (half ? e.dHv : e.dHu);
                eo = sA * (half ? e.dHu : e.dHv);
            } else if (!half) {
                ec = outer(radius_nu(k), psi, lam);
            }
        }
        double diag = fma(cV, ec + tc, 1.0);
        if (emabs) diag = fma(c, sig, diag);
        if (ln < NT) {
            out.sch[ln] = real ? (TRANS ? -c * tc * iV_prev : cV * to) : 0.0;
            out.bco[ln] = real ? (TRANS ? -c * ec * iVn : cV * eo) : 0.0;
            out.g[ln] = real ? A.rhs_sign * z_rhs : 0.0;
            sm.psi[ln] = real ? psi : 0.0;
            sm.dg[ln] = real ? diag : 1.0;
        }
        tc = -eo;                                                      // the next zone becomes the current one
        to = -ec;
        psi = n_psi;
        sig = n_sig;
        lam = n_lam;
        iV_prev = iVc;
        wave_sync();
        const double iT = rcp_cubic(Tz), camp = c * amp;
        load_next(k, zn + dir);
        load_zone(k, zn);
        r_t = r_l;
        r_l = r_b;
        r_b = A.f.r_edge[eb + clampe((half ? zc : zc + 1) + 2 * dir)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int C = 0; C < CN; ++C) {
            const int col = 16 * C + jc;
            double dgv = sm.dg[col], B[T];
#pragma unroll
            for (int u = 0; u < T; ++u) B[u] = 0.0;
            if (nes) {
                const double pcol = sm.psi[col], ek = s_eps[col];
                const double wc = -camp * pcol, w1c = -camp - wc;       // weights of psi and 1 - psi of the column
                double acc = 0.0;
#pragma unroll
                for (int u = 0; u < T; ++u) {
                    const int row = 4 * u + L.a;
                    const double M = exp_nonpos(-fabs(s_eps[row] - ek) * iT, coef);
                    const double P = sP[row * X::W + col], PM = P * M;
                    const double prow = sm.psi[row];
                    const bool up = row > col;
                    if (TRANS) {                                        // row is k, column k'
                        const double Pt = sPt[row * X::W + col], wr = -camp * prow, w1r = -camp - wr;
                        B[u] = fma((up ? w1r : wr) * Pt, M, (up ? wr : w1r) * Pt);
                    } else {                                            // column is k, row k'
                        B[u] = fma(up ? wc : w1c, PM, (up ? w1c : wc) * P);
                    }
                    // sum over k' for k the column: k' is the row either way
                    const double pq = 1.0 - prow;
                    acc = fma(up ? prow : pq, P, acc);
                    acc = fma(up ? pq : prow, PM, acc);
                }
                dgv = fma(camp, mfma4(1.0, acc, 0.0), dgv);
            }
#pragma unroll
            for (int u = 0; u < T; ++u) {
                const double on = (u / 4 == C && L.g == u % 4 && L.a == L.b) ? 1.0 : 0.0;
                out.block[C * T + u][ln] = u / 4 == C ? fma(on, dgv, B[u]) : B[u];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // The second wavefront assembles the zone of the next step while the first eliminates that of this one.
    if (assembles && delay == 0 && (m > 0 || !half)) assemble(0);
    lds_barrier();
    for (int n = 0; n <= m; ++n) {
        const bool mid = n == m;
        if (mid) {                                                     // the outer half hands its last factor over
            if (half && !assembles) {
#pragma unroll
                for (int q = 0; q < T; ++q)
#pragma unroll
                    for (int C = 0; C < CN; ++C) s_C[q][C][lane] = S.get(q, C);
                if (lane < X::W) s_y[lane] = sm.y[lane];
                if (lane == 0) s_bad[1] = guard.bad != 0ull;
            }
            lds_barrier();
        }
        if (assembles) {
            if (n + 1 >= delay && n + 1 < m + (half ? 0 : 1)) assemble(n + 1);
        } else if (n >= delay && !(mid && half)) {
            const int ln = opaque_lane(), jc = ln & 15;
            const TileLane L(ln);
            const ZoneBlock<T>& in = sm.zone[n & 1];
            if (ln < NT) {
                double g = fma(-in.sch[ln], sm.y[ln], in.g[ln]);
                if (mid) g = fma(-in.bco[ln], s_y[ln], g);
                sm.g[ln] = g;
            }
            // ---- Schur term of the previous factor, of both neighbours' in the meeting zone
#pragma unroll
            for (int C = 0; C < CN; ++C) {
                const double sc = -in.sch[16 * C + jc], bc = in.bco[16 * C + jc];
#pragma unroll
                for (int q = 0; q < T; ++q) {
                    S.set(q, C, fma(S.get(q, C), sc, in.block[C * T + q][ln]));
                    if (mid) S.set(q, C, fma(-s_C[q][C][ln], bc, S.get(q, C)));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // ---- Ahat^-1, y = Ahat^-1 g, C = Ahat^-1 diag(b)
            wave_invert<T, CN, X::PR, TRANS>(S, L, jc, sm.pan, guard);
            double yc[CN];
#pragma unroll
            for (int C = 0; C < CN; ++C) yc[C] = 0.0;
#pragma unroll
            for (int q = 0; q < T; ++q) {
                const double g = sm.g[4 * q + L.a];
#pragma unroll
                for (int C = 0; C < CN; ++C) yc[C] = fma(S.get(q, C), g, yc[C]);
            }
#pragma unroll
            for (int C = 0; C < CN; ++C) yc[C] = mfma4(1.0, yc[C], 0.0);
            if (L.a == 0) {
#pragma unroll
                for (int C = 0; C < CN; ++C) sm.y[16 * C + jc] = yc[C];
            }
            wave_sync();
            if (!mid) {
#pragma unroll
                for (int q = 0; q < T; ++q) {
                    const double b = in.bco[4 * q + L.a];
#pragma unroll
                    for (int C = 0; C < CN; ++C) S.set(q, C, S.get(q, C) * b);
                }
                store(n, ln);
            }
        }
        if (!mid) lds_barrier();
    }
    if (wave == 0) {
        if (lane == 0) s_bad[0] = guard.bad != 0ull;
        if (lane < X::W) s_x[lane] = sm.y[lane];
    }
    __syncthreads();
    // a system whose growth guard tripped is left to the pivoting re-run
    const bool bad = s_bad[0] || s_bad[1];
    if (bad) {
        if (threadIdx.x == 0) {
            if (A.guard) A.guard[sys] = 1;
            if (A.flags) A.flags[sys] |= 8;
        }
        return;
    }
    if (assembles) return;

    // ---- back substitution outwards from the meeting zone
    const int lb = opaque_lane(), jc = lb & 15;
    const TileLane L(lb);
    auto put = [&](int z, double d) {
        if (lb < N) {
            const size_t ci = cb + (size_t)z * N + lb;
            if (A.psi_out) {
                A.psi_out[ci] += d;
                if (A.dx) A.dx[ci] = d;
            } else {
                A.x[ci] = d;
            }
        }
    };
    if (lb < X::W) sm.y[lb] = s_x[lb];
    if (!half) put(m, lb < X::W ? s_x[lb] : 0.0);
    wave_sync();
    constexpr int D = 4;                                                // zones in flight
    double Cb[D][T][CN], yb[D][CN];                                      // y in column form
    auto fetch = [&](int n, double (&c_)[T][CN], double (&y_)[CN]) {
        const double* slot = ws + (size_t)(half ? I - 1 - (n - delay) : n) * SZ;
#pragma unroll
        for (int C = 0; C < X::FC; ++C) {
#pragma unroll
            for (int q = 0; q + 1 < T; q += 2) {
                const V2 v = nt_load(reinterpret_cast<const V2*>(slot + 64 * T * C) + 32 * q + lb);
                c_[q][C] = v.x;
                c_[q + 1][C] = v.y;
            }
            if (T & 1) c_[T - 1][C] = nt_load(slot + 64 * T * C + 64 * (T - 1) + lb);
        }
        if constexpr (X::REM > 0) {
#pragma unroll
            for (int q = 0; q < T; ++q)
                c_[q][X::FC] = jc < X::REM ? nt_load(slot + 64 * T * X::FC + 4 * X::REM * q + X::REM * L.a + jc) : 0.0;
        }
#pragma unroll
        for (int C = 0; C < CN; ++C) y_[C] = 16 * C + jc < NT ? nt_load(slot + (size_t)NT * NT + 16 * C + jc) : 0.0;
    };
    auto step = [&](int n, const double (&c_)[T][CN], const double (&y_)[CN]) {
        double acc[CN];
#pragma unroll
        for (int C = 0; C < CN; ++C) acc[C] = 0.0;
#pragma unroll
        for (int q = 0; q < T; ++q) {
            const double x = sm.y[4 * q + L.a];
#pragma unroll
            for (int C = 0; C < CN; ++C) acc[C] = fma(c_[q][C], x, acc[C]);
        }
#pragma unroll
        for (int C = 0; C < CN; ++C) acc[C] = y_[C] - mfma4(1.0, acc[C], 0.0);
        wave_sync();
        if (L.a == 0) {
#pragma unroll
            for (int C = 0; C < CN; ++C) sm.y[16 * C + jc] = acc[C];
        }
        wave_sync();
        put(half ? I - 1 - (n - delay) : n, lb < X::W ? sm.y[lb] : 0.0);
    };
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
        if (m - 1 - d >= delay) fetch(m - 1 - d, Cb[d], yb[d]);
    for (int n = m - 1; n >= delay; n -= D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (n - d < delay) break;
            if (n - d - (D - 1) >= delay) fetch(n - d - (D - 1), Cb[(d + D - 1) % D], yb[(d + D - 1) % D]);
            step(n - d, Cb[d], yb[d]);
        }
    }
    if (threadIdx.x == 0 && A.psi_out) {
        if (A.iters) A.iters[sys] += 1;
        if (A.pending) A.pending[sys] = 1;                              // trial psi + delta awaits the line search
        if (A.alpha) A.alpha[sys] = 1.0;
    }
}

template <int T>
static void launch_single_t(const FactorArgs& a, bool transpose, hipStream_t st) {
    const dim3 grid((unsigned)a.nsys), block(256);
    const bool ext = a.f.lapse || a.sh.limiter == 2 || a.sh.outer_bc == 2;
    if (transpose) {
        if (ext) hipLaunchKernelGGL((k_factor_wave<T, true, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_factor_wave<T, true, false>), grid, block, 0, st, a);
    } else {
        if (ext) hipLaunchKernelGGL((k_factor_wave<T, false, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_factor_wave<T, false, false>), grid, block, 0, st, a);
    }
}

hipError_t launch_factor_wave(const FactorArgs& a, bool transpose, hipStream_t st) {
    switch (padded_groups(a.sh.N)) {
        case 4: launch_single_t<1>(a, transpose, st); break;
        case 8: launch_single_t<2>(a, transpose, st); break;
        case 12: launch_single_t<3>(a, transpose, st); break;
        case 16: launch_single_t<4>(a, transpose, st); break;
        case 20: launch_single_t<5>(a, transpose, st); break;
        case 24: launch_single_t<6>(a, transpose, st); break;
        case 28: launch_single_t<7>(a, transpose, st); break;
        case 32: launch_single_t<8>(a, transpose, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace tmk

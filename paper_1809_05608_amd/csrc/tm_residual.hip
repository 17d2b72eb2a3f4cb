// FP64 kernels of libtm over cells: grid constants, residual with per-system norms and
// conservation sums, debug Jacobian blocks, and the adjoint vector-Jacobian product.
//
// Mapping of the residual and VJP kernels: one block per (species, ray) system, a chunk
// of zones at a time; each edge flux is computed once, and the block reduces per-system quantities
// in a fixed order (deterministic, no atomics).
#include <algorithm>
#include <type_traits>

#include "tm_kernels.hpp"
#include "tm_nes.hpp"

namespace tmk {

// ---------------------------------------------------------------- grid constants

__global__ void k_setup(const double* __restrict__ e_edge, const double* __restrict__ nes_g, int N,
                        Consts* __restrict__ out) {
    __shared__ double eps[kMaxN], W[kMaxN];
    __shared__ double wbar;
    const int t = threadIdx.x;
    if (t < N) {
        const double lo = e_edge[t], hi = e_edge[t + 1];
        eps[t] = sqrt((hi * hi + hi * lo + lo * lo) * (1.0 / 3.0));   // eq. a01, square restored
        W[t] = (hi - lo) * (hi * hi + hi * lo + lo * lo) * (1.0 / 3.0); // eq. a01b
    }
    __syncthreads();
    if (t == 0) {
        double s = 0.0;
        for (int k = 0; k < N; ++k) s += W[k];
        wbar = s / N;
    }
    __syncthreads();
    if (t < kMaxN) {
        out->eps[t] = t < N ? eps[t] : 0.0;
        out->W[t] = t < N ? W[t] : 0.0;
        out->de[t] = (t + 1 < N) ? eps[t + 1] - eps[t] : 0.0;
    }
    if (t == 0) {
        int ok = 1;
        for (int k = 1; k < N; ++k) ok &= eps[k] >= 1.25 * eps[k - 1];
        out->nes_window = ok;
        out->wbar = wbar;
    }
    for (int idx = t; idx < kMaxN * kMaxN; idx += blockDim.x) {
        const int k = idx / kMaxN, kp = idx % kMaxN;
        double v = 0.0;
        // k' = k (no energy change) is left out: its in and out terms cancel identically (eq. d8b)
        if (k < N && kp < N && kp != k && nes_g != nullptr)
            v = eps[k] * eps[kp] / (kEps0 * kEps0) * nes_g[k * N + kp] * (W[kp] / wbar);
        out->P[k][kp] = v;
    }
}

hipError_t launch_setup(const double* e_edge, const double* nes_g, int N, Consts* out, hipStream_t st) {
    hipLaunchKernelGGL(k_setup, dim3(1), dim3(256), 0, st, e_edge, nes_g, N, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- per-zone pieces

// NES source of one zone: S_k = amp [(1 - p_k) sum_k' P Ein p_k' - p_k sum_k' P Eout (1 - p_k')]
// with the detailed-balance factor exp(-|eps_k - eps_k'|/T) built as a product of
// neighbour factors d_j = exp(-(eps_{j+1} - eps_j)/T) (Eout for k' > k, Ein for k' < k).
// Also returns the two kernel sums (without amp) for the Jacobian diagonal.
template <int NT>
__device__ __forceinline__ void nes_zone(const Consts* __restrict__ cs, int N, double T, const double* p,
                                         double* sin_out, double* sout_out) {
    double d[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) d[j] = (j + 1 < N) ? exp(-cs->de[j] / T) : 0.0;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        if (k >= N) break;
        double sin_ = 0.0;
        double sout = 0.0;
        double e = 1.0;
#pragma unroll
        for (int kp = k + 1; kp < NT; ++kp) {          // up-scatter side: out factor decays
            if (kp >= N) break;
            e *= d[kp - 1];
            sout = fma(cs->P[k][kp] * e, 1.0 - p[kp], sout);
            sin_ = fma(cs->P[k][kp], p[kp], sin_);
        }
        e = 1.0;
#pragma unroll
        for (int kp = k - 1; kp >= 0; --kp) {          // down-scatter side: in factor decays
            e *= d[kp];
            sin_ = fma(cs->P[k][kp] * e, p[kp], sin_);
            sout = fma(cs->P[k][kp], 1.0 - p[kp], sout);
        }
        sin_out[k] = sin_;
        sout_out[k] = sout;
    }
}

struct ZoneGeom {
    double V, A_lo, A_hi, D_lo, D_hi, V_lo, V_hi;
};

// Geometry of zone i of a ray; with a lapse (f.lapse set) the volumes are V / a^3 and the areas A / a^2.
__device__ __forceinline__ ZoneGeom zone_geom(const double* __restrict__ re, int i, int I, const Fields& f,
                                              int ray) {
    ZoneGeom g;
    const double rlo = re[i], rhi = re[i + 1];
    const size_t z = (size_t)ray * I + i, e = (size_t)ray * (I + 1) + i;
    g.V = shell_volume(rlo, rhi) / lapse_zone3(f, z);
    g.A_lo = rlo * rlo * lapse_edge_inv2(f, e);
    g.A_hi = rhi * rhi * lapse_edge_inv2(f, e + 1);
    const double rc = 0.5 * (rlo + rhi);
    g.D_lo = 0.0;
    g.V_lo = 1.0;
    g.D_hi = 0.0;
    g.V_hi = 1.0;
    if (i > 0) {
        const double rm = re[i - 1];
        g.D_lo = rc - 0.5 * (rm + rlo);
        g.V_lo = shell_volume(rm, rlo) / lapse_zone3(f, z - 1);
    }
    if (i + 1 < I) {
        const double rp = re[i + 2];
        g.D_hi = 0.5 * (rhi + rp) - rc;
        g.V_hi = shell_volume(rhi, rp) / lapse_zone3(f, z + 1);
    }
    return g;
}

__device__ __forceinline__ double inv_mfp(const Fields& f, size_t c) {
    return 1.0 / (f.kappa_a[c] + f.eta[c] + f.kappa_s[c]);
}

// ---------------------------------------------------------------- residual / statistics

// Mapping: one block per system, its one to four wavefronts taking consecutive parts of the ray, in chunks of 16 zones.
// Lane 16 a + j holds groups a, 4 + a, 8 + a, ... of the chunk's zone j: the natural order of the 4 x 4 x 4
// matrix products with the sixteen zones as columns.  The NES sums over k' are products of the constant shape
// matrix with vectors per zone, so they go to the matrix cores, tile by tile (nes_sums); a neighbouring zone's
// value is one lane away (two DPP moves); LDS holds only the constants.  Each edge flux is computed once, by the
// zone below the edge; a chunk's last row serves as the upper neighbour only, and the flux below its first row
// comes from the chunk before.
// The sums over k' in Horner form, one cell per thread (the kernel by cells below), took 38 steps of three LDS reads (32 bytes a lane) and were
// bound by LDS; now vector issue (61% of the cycles) and memory share the time: 32768 systems of 540 zones x 20
// groups 7.3 -> 4.6 ms (48 bytes a cell once: 3.9 ms at the 4.4 TB/s of a copy), with the geometric options 9.6 ->
// 5.0, 16384 systems of 300 x 32 4.5 -> 2.6, of 300 x 12 1.0 -> 0.9, 720 of 540 x 20 0.26 -> 0.14.  Loading in the
// layout of the sums instead (32-byte pieces, no way through LDS) took 6.1 ms, most of it in the address units; a
// chunk's loads one chunk ahead, at two wavefronts a SIMD instead of three, 5.4.
// Besides max|G| the kernel computes the rounding level of G (32 ulp of the largest per-cell sum of term
// magnitudes plus |psi| |dG/dpsi|), below which the Newton stopping rule does not ask for further progress.

// A value from the neighbouring zone's lane: j + 1 (row 15 gets its own), or j - 1 with `first` in row 0.
__device__ __forceinline__ double zone_up(double v) {
    const long long w = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp((int)w, (int)w, 0x101, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(w >> 32), (int)(w >> 32), 0x101, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double zone_down(double v, double first) {
    const long long w = __double_as_longlong(v), f = __double_as_longlong(first);
    const int lo = __builtin_amdgcn_update_dpp((int)f, (int)w, 0x111, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(f >> 32), (int)(w >> 32), 0x111, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// 1/sqrt(x) from the hardware estimate (about 2^-22) and one cubic step: y + y e (1/2 + 3/8 e), e = 1 - x y^2.
__device__ __forceinline__ double rsqrt_newton(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y, e * fma(e, 0.375, 0.5), y);
}

// Element at a byte offset from a wave-uniform base (scalar base, 32-bit lane offset).
template <typename D>
__device__ __forceinline__ D& at(D* base, unsigned off) {
    return *(D*)((uintptr_t)base + off);
}

// A residual pass's end for one system, by all threads of its block: max|G|, the rounding level, the Newton and
// line-search decisions, the conservation sums.  `bad`: the thread met a G that is not finite.
struct ResidualSums {
    double n = 0.0, nold = 0.0, e = 0.0, q = 0.0, nes = 0.0, b = 0.0;
};
template <int THREADS>
__device__ __forceinline__ void residual_end(const Shape& sh, const Fields& f, const ResidualOut& out, long long sys,
                                             double gmax, double gscale, int bad, ResidualSums s, double* red) {
    const int I = sh.I, ray = (int)(sys % sh.R);
    const double res = block_max<THREADS>(gmax, red);
    const double floor_g = 32.0 * 2.220446049250313e-16 * block_max<THREADS>(gscale, red);
    bad = block_or<THREADS>(bad, red);
    if (out.stats) {
        s.n = block_sum<THREADS>(s.n, red);
        s.nold = block_sum<THREADS>(s.nold, red);
        s.e = block_sum<THREADS>(s.e, red);
        s.q = block_sum<THREADS>(s.q, red);
        s.nes = block_sum<THREADS>(s.nes, red);
        s.b = block_sum<THREADS>(s.b, red);
    }
    if (threadIdx.x == 0) {
        const double rr = bad ? __builtin_nan("") : res;
        out.res[sys] = rr;
        if (out.level) out.level[sys] = floor_g;
        const int it = out.iters ? out.iters[sys] : 0;
        if (out.mode == kResInitial) {
            // Newton stopping rule: max|G| <= target = max(rtol * max|G_0|, rounding level of G), or no
            // halving of max|G| within 1000x of the target; rtol = 0 means a fixed number of updates
            const double target = fmax(out.rtol * rr, floor_g);
            out.res0[sys] = rr;
            out.res_acc[sys] = rr;
            out.tgt[sys] = target;
            const bool stop = out.rtol > 0.0 && !bad && rr <= target;
            out.active[sys] = (!stop && !bad && it < out.max_iter && rr > 0.0) ? 1 : 0;
        } else if (out.mode == kResTrial) {
            // backtracking line search: accept the trial on sufficient decrease of max|G|, at the
            // shortest step, or when the previous iterate was already within 1000x of its target
            const double racc = out.res_acc[sys], a = out.alpha[sys];
            const bool near = racc <= 1e3 * out.tgt[sys];
            const bool accept = near || rr <= (1.0 - kArmijo * a) * racc || a <= kAlphaMin;
            if (accept) {
                const double target = fmax(out.rtol * out.res0[sys], floor_g);
                out.pending[sys] = 0;
                out.backtrack[sys] = 0;
                out.res_acc[sys] = rr;
                out.tgt[sys] = target;
                const bool stop = out.rtol > 0.0 && !bad && (rr <= target || (rr <= 1e3 * target && rr > 0.5 * racc));
                out.active[sys] = (!stop && !bad && it < out.max_iter && rr > 0.0) ? 1 : 0;
            } else {
                out.backtrack[sys] = 1;
            }
        }
        if (out.stats) {
            const double rI = f.r_edge[(size_t)ray * (I + 1) + I], rout = rI * rI * lapse_edge_inv2(f, (size_t)ray * (I + 1) + I);
            const double b = sh.c_dt * rout * s.b;
            if (out.n_tot) out.n_tot[sys] = s.n;
            if (out.e_tot) out.e_tot[sys] = s.e;
            if (out.budget) out.budget[sys] = s.n - s.nold + b - s.q - s.nes;
            if (out.lum) out.lum[sys] = kCLight * rout * s.b;
        }
    }
}

// GEO compiles the neutrinosphere options (limiter 2, outer boundary 2) in; W is the block's number of wavefronts.
template <int T, bool GEO, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(T <= 3 ? 4 : T <= 5 ? 3 : 2)))
void k_residual(Shape sh, Fields f, const Consts* __restrict__ cs, const double* __restrict__ psi_n,
                const double* __restrict__ psi, double* __restrict__ G_out, double g_sign, ResidualOut out) {
    constexpr int NT = 4 * T;
    __shared__ NesLds<T> sm;
    __shared__ double s_W[NT], s_We[NT], s_de[NT], s_rnu[GEO ? NT : 1];
    constexpr int PS = NT + 1;                            // row stride: the 16 rows of a group in different banks
    __shared__ double s_cell[W][4][16 * PS + 1];          // a chunk's psi, then psi_n, then G; kappa_a, eta, kappa_s
    __shared__ double2 s_edge[W][T][4];         // flux and derivative at the edge above row 14
    __shared__ double red[W];
    const long long sys = blockIdx.x;
    if (out.mode == kResTrial && out.pending[sys] == 0) return;         // no trial to evaluate
    if (out.mode == kResEval && out.pending && out.pending[sys % sh.R] == 0) return;
    const int I = sh.I, N = sh.N;
    const int ray = (int)(sys % sh.R);
    const double* re = f.r_edge + (size_t)ray * (I + 1);
    const double c = sh.c_dt;
    const bool diff = sh.terms & kDiffusion, emabs = sh.terms & kEmAbs, nes = sh.terms & kNes;
    const bool geo = GEO && (sh.limiter == 2 || sh.outer_bc == 2);      // neutrinosphere radii in use
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    if (nes) sm.template fill<64 * W>(*cs);
    if (threadIdx.x < NT) {
        const int k = threadIdx.x;
        s_W[k] = k < N ? cs->W[k] : 0.0;
        s_We[k] = k < N ? cs->W[k] * cs->eps[k] : 0.0;
        s_de[k] = k + 1 < N ? cs->de[k] : 0.0;
        if (geo) s_rnu[k] = k < N ? f.r_nu[(size_t)(sys / sh.R) * N + k] : 0.0;
    }
    __syncthreads();

    double gmax = 0.0, gscale = 0.0;
    int bad = 0;
    ResidualSums sums;
    const size_t cells = (size_t)sys * I * N;
    const double* const zT = f.temp ? f.temp + (size_t)ray * I : re;
    const double* const zA = f.nes_amp ? f.nes_amp + (size_t)sys * I : re;

    // this wavefront's zones lo .. hi - 1; row 0 of its first chunk is the zone below them.  Whole chunks, so that no
    // wavefront takes another one for a zone or two: 15 zones each, one of them the zone below but in the first.
    const int per = 15 * ((I + W - 1 + 15 * W - 1) / (15 * W)) - 1;
    const int lo = wave == 0 ? 0 : min(I, wave * per + 1), hi = min(I, (wave + 1) * per + 1);
    if ((threadIdx.x & 63) < 4 * T)                      // the edge below zone 0 has zero flux
        s_edge[wave][(threadIdx.x & 63) >> 2][threadIdx.x & 3] = make_double2(0.0, 0.0);
    const int zf = lo == hi ? hi : lo > 0 ? lo - 1 : 0;
    const float iN = 1.0f / (float)N;
    for (int z0 = zf; z0 < hi; z0 += 15) {
        // what derives from the lane id, the constants in LDS among it, is fetched again for each chunk
        const int lane = opaque_lane(), a = lane >> 4, j = lane & 15, b = lane & 3, ab = 4 * a + b;
        const int i = z0 + j, ic = min(i, I - 1);
        int lo_v = lo, hi_v = hi;                             // in vector registers: the geometric options spill scalars
        if (GEO) asm volatile("" : "+v"(lo_v), "+v"(hi_v));
        const bool out_row = j < 15 && i >= lo_v && i < hi_v;
        // a chunk's cells are contiguous: loaded and stored in order, turned into zones by groups in LDS
        const size_t chunk = cells + (size_t)z0 * N;
        const int last = min(16, I - z0) * N - 1;
        double nx[5][T];
#pragma unroll
        for (int q = 0; q < T; ++q) {
            const unsigned o = 8u * (unsigned)min(64 * q + lane, last);
            nx[0][q] = at(psi + chunk, o);
            nx[1][q] = at(f.kappa_a + chunk, o);
            nx[2][q] = at(f.eta + chunk, o);
            nx[3][q] = at(f.kappa_s + chunk, o);
            nx[4][q] = at(psi_n + chunk, o);
        }
        auto slot = [&](int q) {                              // of cell 64 q + lane: row x / N, group x % N
            const int x = 64 * q + lane, row = (int)(((float)x + 0.5f) * iN);
            return row < 16 ? row * PS + x - row * N : 16 * PS;      // past the chunk: one spare element
        };
#pragma unroll
        for (int q = 0; q < T; ++q) {
            const int o = slot(q);
#pragma unroll
            for (int v = 0; v < 4; ++v) s_cell[wave][v][o] = nx[v][q];
        }
        const double rlo = re[ic], rhi = re[ic + 1], rp = re[min(ic + 2, I)];
        const double amp = nes ? zA[ic] : 0.0, Tz = nes ? zT[ic] : 1.0;
        wave_sync();
        double p[T];                                          // padding groups repeat the last one
#pragma unroll
        for (int t = 0; t < T; ++t) p[t] = s_cell[wave][0][j * PS + (t + 1 < T ? 4 * t + a : min(4 * t + a, N - 1))];
        wave_sync();
#pragma unroll
        for (int q = 0; q < T; ++q) s_cell[wave][0][slot(q)] = nx[4][q];
        wave_sync();
        double sin_[T], sout[T];
        if (nes) {
            const double iT = drcp(Tz);
            const ExpCoef coef = exp_coef();
            double d[T];
#pragma unroll
            for (int t = 0; t < T; ++t) d[t] = exp_nonpos(-s_de[4 * t + a] * iT, coef);
            nes_sums<T>(sm, p, d, a, b, ab, sin_, sout);
        }
        double V = shell_volume(rlo, rhi), A_lo = rlo * rlo, A_hi = rhi * rhi;
        if (f.lapse) {                                      // eq. a58 times a_i c dt: V / a^3 and A / a^2
            const double a0 = f.lapse[(size_t)ray * I + ic];
            const double e0 = f.lapse_edge[(size_t)ray * (I + 1) + ic], e1 = f.lapse_edge[(size_t)ray * (I + 1) + ic + 1];
            V /= a0 * a0 * a0;
            A_lo /= e0 * e0;
            A_hi /= e1 * e1;
        }
        const double iV = drcp(V), D = 0.5 * (rhi + rp) - 0.5 * (rlo + rhi);
        double w_n = 0.0, w_old = 0.0, w_e = 0.0, w_q = 0.0, w_nes = 0.0;    // the zone's sums over its groups
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int k = 4 * t + a;
            const bool ok = t + 1 < T ? out_row : out_row && k < N;
            __builtin_amdgcn_sched_barrier(0);
            const int o = j * PS + 4 * t + a;
            const double ka = s_cell[wave][1][o], et = s_cell[wave][2][o], ks = s_cell[wave][3][o], pn = s_cell[wave][0][o];
            const double h = 1.0 - p[t], sig = ka + et;
            double H = 0.0, du = 0.0, dv = 0.0, H_lo = 0.0, d_lo = 0.0;
            if (diff) {
                const double chi = sig + ks;
                const double p_up = zone_up(p[t]), chi_up = zone_up(chi);
                const double rnu = geo ? s_rnu[k] : 0.0;
                if (i + 1 < I) {                            // mean free path at the edge: geometric mean
                    const EdgeFlux e = edge_flux(p[t], p_up, rsqrt_newton(chi * chi_up), D, sh.psi_floor, sh.limiter,
                                                 (GEO && sh.limiter == 2) ? limb_factor(rhi, rnu) : -1.0);
                    H = e.H;
                    du = e.dHu;
                    dv = e.dHv;
                } else if (sh.outer_bc == 1) {
                    H = p[t];                               // free streaming, eq. a22 limit
                    du = 1.0;
                } else if (GEO && sh.outer_bc == 2) {       // ghost zone of eq. a62af
                    const Ghost gh = outer_ghost(rlo, rhi, rnu);
                    const EdgeFlux e = edge_flux(p[t], gh.ratio * p[t], drcp(chi), gh.D, sh.psi_floor, sh.limiter,
                                                 sh.limiter == 2 ? limb_factor(rhi, rnu) : -1.0);
                    H = e.H;
                    du = e.dHu + gh.ratio * e.dHv;
                }
                const double2 below = s_edge[wave][t][a];
                H_lo = zone_down(H, below.x);
                d_lo = zone_down(dv, below.y);
                wave_sync();
                if (j == 14) s_edge[wave][t][a] = make_double2(H, dv);
            }
            if (!ok) continue;
            // G = psi - psi_n + c dt (rest); size: the same sum of magnitudes; jd: |dG_ik/dpsi_ik| bound
            double rest = 0.0, size = 0.0, jd = 0.0;
            if (diff) {
                const double up = A_hi * H, dn = A_lo * H_lo;
                rest = (up - dn) * iV;
                size = (fabs(up) + fabs(dn)) * iV;
                jd = (A_hi * fabs(du) + A_lo * fabs(d_lo)) * iV;
            }
            double em = 0.0;
            if (emabs) {
                const double ab = ka * p[t], re_ = et * h;
                em = ab - re_;
                rest += em;
                size += fabs(ab) + fabs(re_);
                jd += sig;
            }
            double S = 0.0;
            if (nes) {
                const double in = h * sin_[t], ex = p[t] * sout[t];
                S = in - ex;
                rest = fma(-amp, S, rest);
                size = fma(amp, fabs(in) + fabs(ex), size);
                jd = fma(amp, fabs(sin_[t]) + fabs(sout[t]), jd);
            }
            const double G = fma(c, rest, p[t] - pn);
            const double scale = fma(c, size, fabs(p[t]) + fabs(pn)) + fabs(p[t]) * fma(c, jd, 1.0);  // G per ulp of psi
            bad |= !isfinite(G);
            gmax = fmax(gmax, fabs(G));
            gscale = fmax(gscale, scale);
            s_cell[wave][0][o] = g_sign * G;
            if (out.stats) {
                const double Wk = s_W[k];
                w_n = fma(Wk, p[t], w_n);
                w_old = fma(Wk, pn, w_old);
                w_e = fma(s_We[k], p[t], w_e);
                w_q = fma(Wk, em, w_q);
                w_nes = fma(Wk, S, w_nes);
                if (i == I - 1 && diff) sums.b = fma(Wk, H, sums.b);
            }
        }
        if (out.stats && out_row) {
            sums.n = fma(V, w_n, sums.n);
            sums.nold = fma(V, w_old, sums.nold);
            sums.e = fma(V, w_e, sums.e);
            sums.q = fma(-c * V, w_q, sums.q);
            sums.nes = fma(c * V * amp, w_nes, sums.nes);
        }
        wave_sync();
        if (G_out) {
            const int x0 = (max(z0, lo_v) - z0) * N, x1 = (min(z0 + 15, hi_v) - z0) * N;      // the rows put out
#pragma unroll
            for (int q = 0; q < T; ++q) {
                const int x = 64 * q + lane;
                if (x >= x0 && x < x1) at(G_out + chunk, 8u * (unsigned)x) = s_cell[wave][0][slot(q)];
            }
        }
        wave_sync();
    }

    residual_end<64 * W>(sh, f, out, sys, gmax, gscale, bad, sums, red);
}

// Up to four groups a zone is a single column of the matrix products above, a quarter to all of it padding, and a
// chunk's way through LDS and the sums of products cost more than they save; on rays of a few zones most of a chunk's
// sixteen are padding, and a wavefront works through their groups alone.  There a thread is a cell.  The 256 threads
// form 256 / NT rows of NT groups; row r of a chunk holds zone z0 - 1 + r, and the first and the last row are halo.
// Every cell brings psi and its mean free path to LDS, computes the flux at its upper edge, and then G from both fluxes
// of its zone and the scattering sums over the zone's row, in Horner form.  The next chunk's loads are in flight while
// a chunk is worked on.  Latency and LDS bound it.  100 zones, against the sixteen-zone chunks above: 65536 systems
// of one group 0.45 against 0.55 ms, of four 0.52 against 0.60; 256 systems of four 19.9 against 21.5 us.
// LAPSE and GEO compile the lapse factors and the neutrinosphere options in.
template <int NT, bool LAPSE, bool GEO>
__global__ __launch_bounds__(kBlock) void k_residual_rows(Shape sh, Fields f, const Consts* __restrict__ cs,
                                                          const double* __restrict__ psi_n,
                                                          const double* __restrict__ psi, double* __restrict__ G_out,
                                                          double g_sign, ResidualOut out) {
    constexpr int RZ = kBlock / NT;             // rows per chunk (zones incl. one halo on each side)
    constexpr int ZB = RZ - 2;                  // output zones per chunk
    constexpr int PS = NT + 1;                  // padded LDS row stride (conflict-free column reads)
    static_assert(3 * RZ + 2 <= kBlock, "one zone value per thread");
    __shared__ double s_P[NT * PS];
    __shared__ double s_psi[RZ][PS];
    __shared__ double2 s_pq[RZ][NT];            // psi and 1 - psi of the row (the NES sums read both at once)
    __shared__ double s_lam[RZ][PS];
    __shared__ double s_d[RZ][PS];
    __shared__ double s_H[RZ][PS];              // flux at the upper edge of the row's zone
    __shared__ double s_du[RZ][PS];             // its derivative with respect to the lower zone
    __shared__ double s_dv[RZ][PS];             // ... and to the upper zone
    __shared__ double s_z[3 * RZ + 2];          // edges z0-1 .. z0+RZ, then T and amp of the rows
    __shared__ double red[kBlock / 64];
    double* const s_re = s_z;
    double* const s_T = s_z + RZ + 2;
    double* const s_amp = s_z + 2 * RZ + 2;
    const long long sys = blockIdx.x;
    if (out.mode == kResTrial && out.pending[sys] == 0) return;         // no trial to evaluate
    if (out.mode == kResEval && out.pending && out.pending[sys % sh.R] == 0) return;
    const int I = sh.I, N = sh.N;
    const int ray = (int)(sys % sh.R);
    const double* re = f.r_edge + (size_t)ray * (I + 1);
    const double c = sh.c_dt;
    const bool diff = sh.terms & kDiffusion, emabs = sh.terms & kEmAbs, nes = sh.terms & kNes;
    const int t = threadIdx.x, zl = t / NT, k = t - zl * NT;
    const bool tile = zl < RZ;                  // a row of the chunk: not the remainder of 256 threads by NT
    const bool lane_ok = tile && k < N;
    const bool out_row = zl >= 1 && zl <= RZ - 2;

    if (nes)
        for (int j = t; j < NT * NT; j += kBlock) s_P[(j / NT) * PS + (j % NT)] = cs->P[j / NT][j % NT];

    double gmax = 0.0, gscale = 0.0;
    int bad = 0;
    ResidualSums sums;
    const double Wk = lane_ok ? cs->W[k] : 0.0;
    const double epsk = lane_ok ? cs->eps[k] : 0.0;
    const bool geo = GEO && (sh.limiter == 2 || sh.outer_bc == 2);   // neutrinosphere radii in use
    const double rnuk = (geo && lane_ok) ? f.r_nu[(size_t)(sys / sh.R) * N + k] : 0.0;
    const double dek = (lane_ok && k + 1 < N) ? cs->de[k] : 0.0;
    const size_t sys_cell0 = (size_t)sys * I * N;

    // per-thread inputs of one chunk: the cell's fields and one zone value
    struct In {
        double p, ka, et, ks, pn, zv;
    };
    // Every load is issued unconditionally from a clamped, in-bounds address and the value selected
    // afterwards: straight-line code lets the wait for a chunk's data count exactly the loads
    // issued after it, instead of draining the memory pipe.
    auto load = [&](int z0, In& v) {
        const int i = z0 - 1 + zl;
        const bool in_zone = lane_ok && i >= 0 && i < I;
        const bool outc = in_zone && out_row;
        const size_t cb = sys_cell0 + (in_zone ? (size_t)i * N + k : 0);
        const double lp = psi[cb], lka = f.kappa_a[cb], let = f.eta[cb], lks = f.kappa_s[cb], lpn = psi_n[cb];
        const bool opac = diff ? in_zone : (emabs && outc);
        v.p = (diff ? in_zone : outc) ? lp : 0.0;
        v.ka = opac ? lka : 0.0;
        v.et = opac ? let : 0.0;
        v.ks = (diff && in_zone) ? lks : 0.0;
        v.pn = outc ? lpn : 0.0;
        const double* src = re;
        bool zok = false;
        double zdef = 0.0;
        if (t < RZ + 2) {
            const int j = z0 - 1 + t;
            zok = j >= 0 && j <= I;
            src = re + (zok ? j : 0);
        } else if (t < 2 * RZ + 2) {
            const int j = z0 - 1 + (t - RZ - 2);
            zok = nes && j >= 0 && j < I;
            src = zok ? f.temp + (size_t)ray * I + j : re;
            zdef = 1.0;
        } else if (t < 3 * RZ + 2) {
            const int j = z0 - 1 + (t - 2 * RZ - 2);
            zok = nes && j >= 0 && j < I;
            src = zok ? f.nes_amp + (size_t)sys * I + j : re;
        }
        const double lz = *src;
        v.zv = zok ? lz : zdef;
    };

    In cur;
    load(0, cur);
    for (int z0 = 0; z0 < I; z0 += ZB) {
        In nxt;
        load(z0 + ZB, nxt);                                 // in flight while this chunk is processed
        const int i = z0 - 1 + zl;                          // this row's zone (may be a halo or outside)
        const bool in_zone = lane_ok && i >= 0 && i < I;
        const double p = cur.p;
        const double lam = (diff && in_zone) ? drcp(cur.ka + cur.et + cur.ks) : 0.0;
        __syncthreads();                                    // previous chunk done with the LDS rows
        if (tile) {
            s_psi[zl][k] = p;
            if (nes) s_pq[zl][k] = make_double2(p, 1.0 - p);
            s_lam[zl][k] = lam;
        }
        if (t < 3 * RZ + 2) s_z[t] = cur.zv;
        __syncthreads();
        if (tile) {
            s_d[zl][k] = (nes && in_zone && out_row && k + 1 < N) ? exp(-dek * drcp(s_T[zl])) : 0.0;
            // flux at the upper edge of this row's zone, computed once per edge
            if (diff) {
                double H = 0.0, du = 0.0, dv = 0.0;
                if (in_zone && zl + 1 < RZ) {
                    if (i + 1 < I) {
                        const double rlo = s_re[zl], rhi = s_re[zl + 1], rp = s_re[zl + 2];
                        const double D = 0.5 * (rhi + rp) - 0.5 * (rlo + rhi);
                        const EdgeFlux e = edge_flux(p, s_psi[zl + 1][k], sqrt(lam * s_lam[zl + 1][k]), D,
                                                     sh.psi_floor, sh.limiter,
                                                     (GEO && sh.limiter == 2) ? limb_factor(rhi, rnuk) : -1.0);
                        H = e.H;
                        du = e.dHu;
                        dv = e.dHv;
                    } else if (sh.outer_bc == 1) {
                        H = p;                              // free streaming, eq. a22 limit
                        du = 1.0;
                    } else if (GEO && sh.outer_bc == 2) {   // ghost zone of eq. a62af
                        const double rlo = s_re[zl], rhi = s_re[zl + 1];
                        const Ghost gh = outer_ghost(rlo, rhi, rnuk);
                        const EdgeFlux e = edge_flux(p, gh.ratio * p, lam, gh.D, sh.psi_floor, sh.limiter,
                                                     sh.limiter == 2 ? limb_factor(rhi, rnuk) : -1.0);
                        H = e.H;
                        du = e.dHu + gh.ratio * e.dHv;
                    }
                }
                s_H[zl][k] = H;                             // the edge below zone 0 has zero flux
                s_du[zl][k] = du;
                s_dv[zl][k] = dv;
            }
        }
        __syncthreads();
        const In now = cur;
        cur = nxt;
        if (!in_zone || !out_row) continue;

        const size_t cb = sys_cell0 + (size_t)i * N + k;
        const double pn = now.pn;
        double G = p - pn;
        double scale = fabs(p) + fabs(pn);
        const double rlo = s_re[zl], rhi = s_re[zl + 1];
        double V = shell_volume(rlo, rhi);
        double A_lo = rlo * rlo, A_hi = rhi * rhi;
        if (LAPSE && f.lapse) {                             // eq. a58 times a_i c dt: V / a^3 and A / a^2
            const double a0 = f.lapse[(size_t)ray * I + i];
            const double e0 = f.lapse_edge[(size_t)ray * (I + 1) + i], e1 = f.lapse_edge[(size_t)ray * (I + 1) + i + 1];
            V /= a0 * a0 * a0;
            A_lo /= e0 * e0;
            A_hi /= e1 * e1;
        }
        double Hh = 0.0;
        double jd = 1.0;                                    // |dG_ik/dpsi_ik| bound, for the rounding level
        if (diff) {
            const double Hlo = s_H[zl - 1][k], dlo = s_dv[zl - 1][k];
            Hh = s_H[zl][k];
            const double dhi = s_du[zl][k];
            const double iV = drcp(V);
            G += c * (A_hi * Hh - A_lo * Hlo) * iV;
            scale += c * (fabs(A_hi * Hh) + fabs(A_lo * Hlo)) * iV;
            jd += c * (A_hi * fabs(dhi) + A_lo * fabs(dlo)) * iV;
        }
        const double ka = now.ka, et = now.et;
        if (emabs) {
            G += c * (ka * p - et * (1.0 - p));
            scale += c * (fabs(ka * p) + fabs(et * (1.0 - p)));
            jd += c * (ka + et);
        }
        double S = 0.0;
        if (nes) {
            const double amp = s_amp[zl];
            // k' > k: the out kernel carries exp(-(eps_k' - eps_k)/T) = prod_{j=k}^{k'-1} d_j.  The weighted sum
            // of those products is taken in Horner form from the last group down, one multiply-add and one
            // multiply per term: h <- (h + P_kk' (1 - psi_k')) d_{k'-1}.
            // The group index through an opaque copy: its compares, one a term, stay inside the zone loop instead of
            // being kept across it as 2 (NT - 1) lane masks.
            int kz = k;
            asm volatile("" : "+v"(kz));
            double hup = 0.0, sin_ = 0.0;
#pragma unroll
            for (int kp = NT - 1; kp >= 1; --kp) {
                if (kp > kz) {                         // padding groups add exact zeros (P = 0 there)
                    const double Pk = s_P[k * PS + kp];
                    const double2 pq = s_pq[zl][kp];
                    hup = fma(Pk, pq.y, hup) * s_d[zl][kp - 1];
                    sin_ = fma(Pk, pq.x, sin_);
                }
            }
            // k' < k: the in kernel carries exp(-(eps_k - eps_k')/T) = prod_{j=k'}^{k-1} d_j, in Horner form from
            // group 0 up: h <- (h + P_kk' psi_k') d_k'
            double hdn = 0.0, sout = hup;
#pragma unroll
            for (int kp = 0; kp < NT - 1; ++kp) {
                if (kp < kz) {
                    const double Pk = s_P[k * PS + kp];
                    const double2 pq = s_pq[zl][kp];
                    hdn = fma(Pk, pq.x, hdn) * s_d[zl][kp];
                    sout = fma(Pk, pq.y, sout);
                }
            }
            sin_ += hdn;
            S = amp * ((1.0 - p) * sin_ - p * sout);
            G -= c * S;
            scale += c * amp * (fabs(1.0 - p) * fabs(sin_) + fabs(p) * fabs(sout));
            jd += c * amp * (fabs(sin_) + fabs(sout));
        }
        scale += fabs(p) * jd;                              // G changes by jd * ulp(psi) per ulp of psi
        bad |= !isfinite(G);
        gmax = fmax(gmax, fabs(G));
        gscale = fmax(gscale, scale);
        if (G_out) G_out[cb] = g_sign * G;
        if (out.stats) {
            const double vw = V * Wk;
            sums.n = fma(vw, p, sums.n);
            sums.nold = fma(vw, pn, sums.nold);
            sums.e = fma(vw * epsk, p, sums.e);
            if (emabs) sums.q = fma(c * vw, et * (1.0 - p) - ka * p, sums.q);
            if (nes) sums.nes = fma(c * vw, S, sums.nes);
            if (i == I - 1 && diff) sums.b = fma(Wk, Hh, sums.b);
        }
    }

    residual_end<kBlock>(sh, f, out, sys, gmax, gscale, bad, sums, red);
}

// ---------------------------------------------------------------- debug Jacobian blocks

template <int NT>
__global__ __launch_bounds__(kBlock) void k_blocks(Shape sh, Fields f, const Consts* __restrict__ cs,
                                                   const double* __restrict__ psi, double* __restrict__ blocks) {
    const long long sys = blockIdx.x;
    const int I = sh.I, N = sh.N;
    const int ray = (int)(sys % sh.R);
    const double* re = f.r_edge + (size_t)ray * (I + 1);
    const double c = sh.c_dt;
    for (int i = threadIdx.x; i < I; i += kBlock) {
        const size_t cb = ((size_t)sys * I + i) * N;
        const ZoneGeom g = zone_geom(re, i, I, f, ray);
        double p[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k) p[k] = k < N ? psi[cb + k] : 0.0;
        double si[NT], so[NT];
        double amp = 0.0;
        const bool nes = sh.terms & kNes;
        if (nes) {
            amp = f.nes_amp[(size_t)sys * I + i];
            nes_zone<NT>(cs, N, f.temp[(size_t)ray * I + i], p, si, so);
        }
        double d[NT];
        if (nes) {
#pragma unroll
            for (int j = 0; j < NT; ++j) d[j] = (j + 1 < N) ? exp(-cs->de[j] / f.temp[(size_t)ray * I + i]) : 0.0;
        }
        for (int k = 0; k < N; ++k) {
            double* row = blocks + (cb + k) * (size_t)(N + 2);
            double diag = 1.0, bm = 0.0, bp = 0.0;
            if (sh.terms & kDiffusion) {
                const double lam = inv_mfp(f, cb + k);
                const double rnu = (sh.limiter == 2 || sh.outer_bc == 2) ? f.r_nu[(size_t)(sys / sh.R) * N + k] : 0.0;
                auto limb = [&](double R) { return sh.limiter == 2 ? limb_factor(R, rnu) : -1.0; };
                double dHv_lo = 0.0, dHu_lo = 0.0, dHu_hi = 0.0, dHv_hi = 0.0;
                if (i > 0) {
                    const size_t cm = cb - N + k;
                    const EdgeFlux e = edge_flux(psi[cm], p[k], sqrt(lam * inv_mfp(f, cm)), g.D_lo,
                                                 sh.psi_floor, sh.limiter, limb(re[i]));
                    dHu_lo = e.dHu;
                    dHv_lo = e.dHv;
                }
                if (i + 1 < I) {
                    const size_t cp = cb + N + k;
                    const EdgeFlux e = edge_flux(p[k], psi[cp], sqrt(lam * inv_mfp(f, cp)), g.D_hi,
                                                 sh.psi_floor, sh.limiter, limb(re[i + 1]));
                    dHu_hi = e.dHu;
                    dHv_hi = e.dHv;
                } else if (sh.outer_bc == 1) {
                    dHu_hi = 1.0;
                } else if (sh.outer_bc == 2) {
                    const Ghost gh = outer_ghost(re[i], re[i + 1], rnu);
                    const EdgeFlux e = edge_flux(p[k], gh.ratio * p[k], lam, gh.D, sh.psi_floor, sh.limiter,
                                                 limb(re[i + 1]));
                    dHu_hi = e.dHu + gh.ratio * e.dHv;
                }
                diag += c * (g.A_hi * dHu_hi - g.A_lo * dHv_lo) / g.V;
                bp = (i + 1 < I) ? c * g.A_hi * dHv_hi / g.V : 0.0;
                bm = (i > 0) ? -c * g.A_lo * dHu_lo / g.V : 0.0;
            }
            if (sh.terms & kEmAbs) diag += c * (f.eta[cb + k] + f.kappa_a[cb + k]);
            const double pk = p[k];
            for (int kp = 0; kp < N; ++kp) {
                double v = 0.0;
                if (nes) {
                    // detailed-balance factor exp(-|eps_k - eps_k'|/T) as a neighbour product
                    double e = 1.0;
                    for (int j = min(k, kp); j < max(k, kp); ++j) e *= d[j];
                    const double kout = amp * cs->P[k][kp] * (kp > k ? e : 1.0);
                    const double kin = amp * cs->P[k][kp] * (kp < k ? e : 1.0);
                    v = -c * ((1.0 - pk) * kin + pk * kout);
                }
                row[kp] = v;
            }
            if (nes) diag += c * amp * (si[k] + so[k]);
            row[k] += diag;
            row[N] = bm;
            row[N + 1] = bp;
        }
    }
}

// ---------------------------------------------------------------- adjoint VJP

template <int NT>
__global__ __launch_bounds__(kBlock) void k_vjp(Shape sh, Fields f, const Consts* __restrict__ cs,
                                                const double* __restrict__ psi, const double* __restrict__ mu,
                                                double* g_ka, double* g_eta, double* g_ks, double* g_amp) {
    // one block per system, one thread per cell: rows of NT threads are zones, so a wave's loads of a
    // cell array (and of the neighbouring zones' cells) are contiguous
    constexpr int RZ = kBlock / NT;             // zones per chunk
    constexpr int PS = NT + 1;                  // padded LDS row stride
    __shared__ double s_P[NT * PS];
    __shared__ double s_p[RZ][PS];              // the zone's psi row
    __shared__ double s_d[RZ][PS];              // neighbour detailed-balance factors exp(-(eps_k+1 - eps_k)/T)
    __shared__ double s_m[RZ][PS];              // mu_k c dt
    __shared__ double s_s[RZ][PS];              // (1 - psi_k) S^in_k - psi_k S^out_k
    const long long sys = blockIdx.x;
    const int I = sh.I, N = sh.N;
    const int ray = (int)(sys % sh.R);
    const double* re = f.r_edge + (size_t)ray * (I + 1);
    const double c = sh.c_dt;
    const bool diff = sh.terms & kDiffusion, emabs = sh.terms & kEmAbs, nes = sh.terms & kNes;
    const bool amp = g_amp != nullptr;
    const int t = threadIdx.x, zl = t / NT, k = t - zl * NT;
    const bool tile = zl < RZ;
    const bool lane_ok = tile && k < N;
    if (amp && nes)
        for (int j = t; j < NT * NT; j += kBlock) s_P[(j / NT) * PS + (j % NT)] = cs->P[j / NT][j % NT];

    for (int z0 = 0; z0 < I; z0 += RZ) {
        const int i = z0 + zl;
        const bool in_zone = lane_ok && i < I;
        const size_t cb = ((size_t)sys * I + (in_zone ? i : 0)) * N + (in_zone ? k : 0);
        double pk = 0.0, m0 = 0.0;
        if (in_zone) {
            const ZoneGeom g = zone_geom(re, i, I, f, ray);
            pk = psi[cb];
            m0 = mu[cb];
            const double lam = inv_mfp(f, cb);
            double gchi = 0.0;     // sum over the two edges of (mu-weighted dG/dH) dH/dlam dlam/dchi
            if (diff) {
                const double rnu = (sh.limiter == 2 || sh.outer_bc == 2) ? f.r_nu[(size_t)(sys / sh.R) * N + k] : 0.0;
                auto limb = [&](double R) { return sh.limiter == 2 ? limb_factor(R, rnu) : -1.0; };
                if (i + 1 < I) {
                    const size_t cp = cb + N;
                    const double lam_e = sqrt(lam * inv_mfp(f, cp));
                    const EdgeFlux e = edge_flux(pk, psi[cp], lam_e, g.D_hi, sh.psi_floor, sh.limiter, limb(re[i + 1]));
                    const double w = c * g.A_hi * (m0 / g.V - mu[cp] / g.V_hi);
                    gchi += w * e.dHlam * (-0.5 * lam_e * lam);
                } else if (sh.outer_bc == 2) {
                    // the ghost-zone flux carries the last zone's own mean free path: dlam/dchi = -lam^2
                    const Ghost gh = outer_ghost(re[i], re[i + 1], rnu);
                    const EdgeFlux e = edge_flux(pk, gh.ratio * pk, lam, gh.D, sh.psi_floor, sh.limiter, limb(re[i + 1]));
                    gchi += c * g.A_hi * (m0 / g.V) * e.dHlam * (-lam * lam);
                }
                if (i > 0) {
                    const size_t cm = cb - N;
                    const double lam_e = sqrt(lam * inv_mfp(f, cm));
                    const EdgeFlux e = edge_flux(psi[cm], pk, lam_e, g.D_lo, sh.psi_floor, sh.limiter, limb(re[i]));
                    const double w = c * g.A_lo * (mu[cm] / g.V_lo - m0 / g.V);
                    gchi += w * e.dHlam * (-0.5 * lam_e * lam);
                }
            }
            // with a lapse the fields are lapse-folded (a kappa_a, a eta, and kappa_s carrying the rest of the
            // transport opacity): the gradient with respect to the caller's kappa_a and eta is a times that
            // with respect to the folded ones plus (1 - a) times the kappa_s one, i.e. the sources carry a
            const double az = f.lapse ? f.lapse[(size_t)ray * I + i] : 1.0;
            double gka = gchi, geta = gchi;
            if (emabs) {
                gka += az * m0 * c * pk;
                geta -= az * m0 * c * (1.0 - pk);
            }
            if (g_ka) g_ka[cb] = -gka;
            if (g_eta) g_eta[cb] = -geta;
            if (g_ks) g_ks[cb] = -gchi;
        }
        if (!amp) continue;
        if (nes) {
            // sum_k mu_k c [(1 - psi_k) S^in_k - psi_k S^out_k] over each zone (the NES source of the zone,
            // Phi_0 terms of eq. d8, differentiated with respect to its amplitude)
            __syncthreads();                                // previous chunk done with the rows
            if (tile) {
                s_p[zl][k] = pk;
                s_d[zl][k] = (in_zone && k + 1 < N) ? exp(-cs->de[k] / f.temp[(size_t)ray * I + i]) : 0.0;
            }
            __syncthreads();
            double s1 = 0.0;
            if (in_zone) {
                double sin_ = 0.0, sout = 0.0, e = 1.0;
                for (int kp = k + 1; kp < N; ++kp) {        // up-scatter side: out factor decays
                    e *= s_d[zl][kp - 1];
                    const double pp = s_p[zl][kp], P = s_P[k * PS + kp];
                    sout = fma(P * e, 1.0 - pp, sout);
                    sin_ = fma(P, pp, sin_);
                }
                e = 1.0;
                for (int kp = k - 1; kp >= 0; --kp) {       // down-scatter side: in factor decays
                    e *= s_d[zl][kp];
                    const double pp = s_p[zl][kp], P = s_P[k * PS + kp];
                    sin_ = fma(P * e, pp, sin_);
                    sout = fma(P, 1.0 - pp, sout);
                }
                s1 = (1.0 - pk) * sin_ - pk * sout;
            }
            if (tile) {
                s_m[zl][k] = m0 * c;
                s_s[zl][k] = s1;
            }
            __syncthreads();
            if (tile && k == 0 && i < I) {
                double ga = 0.0;
                for (int kk = 0; kk < N; ++kk) ga = fma(s_m[zl][kk], s_s[zl][kk], ga);
                // the folded amplitude is amp / a: the caller's amplitude gets 1/a of its gradient
                g_amp[(size_t)sys * I + i] = f.lapse ? ga / f.lapse[(size_t)ray * I + i] : ga;
            }
        } else if (tile && k == 0 && i < I) {
            g_amp[(size_t)sys * I + i] = 0.0;
        }
    }
}

// ---------------------------------------------------------------- lapse folding

// With a lapse the emission/absorption and NES sources of eq. a58 (times a_i c dt) carry a_i, and the NES
// kernels are evaluated at the local energies E / a_i.  Both are exact transformations of the inputs:
// kappa_a -> a kappa_a and eta -> a eta, with kappa_s -> kappa_s + (1 - a)(kappa_a + eta) so that the
// transport mean free path 1/(kappa_a + eta + kappa_s) is unchanged; the NES kernel's energy factor
// eps_k eps_k' / eps0^2 becomes 1/a^2 of its value at infinity and its exponent (eps_k' - eps_k)/T becomes
// (eps_k' - eps_k)/(a T), so amp -> amp / a (with the source's a) and T -> a T.
__global__ __launch_bounds__(kBlock) void k_lapse_fold(long long ncell, int N, long long RI, long long nsz,
                                                       const double* __restrict__ lapse,
                                                       const double* __restrict__ ka, const double* __restrict__ et,
                                                       const double* __restrict__ ks, const double* __restrict__ temp,
                                                       const double* __restrict__ amp, double* __restrict__ oka,
                                                       double* __restrict__ oet, double* __restrict__ oks,
                                                       double* __restrict__ otemp, double* __restrict__ oamp) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < ncell; c += stride) {
        const double a = lapse[(c / N) % RI];
        const double k_a = ka[c], e = et[c];
        oka[c] = a * k_a;
        oet[c] = a * e;
        oks[c] = ks[c] + (1.0 - a) * (k_a + e);
    }
    for (long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x; j < nsz; j += stride) {
        const long long z = j % RI;
        if (amp) oamp[j] = amp[j] / lapse[z];
        if (temp && j < RI) otemp[j] = lapse[j] * temp[j];
    }
}

hipError_t launch_lapse_fold(const Shape& sh, const double* lapse, const double* ka, const double* et,
                             const double* ks, const double* temp, const double* amp, double* oka, double* oet,
                             double* oks, double* otemp, double* oamp, hipStream_t st) {
    const long long RI = (long long)sh.R * sh.I, nsz = (long long)sh.S * RI, ncell = nsz * sh.N;
    const long long blocks = std::min<long long>((ncell + kBlock - 1) / kBlock, 65536);
    hipLaunchKernelGGL(k_lapse_fold, dim3((unsigned)blocks), dim3(kBlock), 0, st, ncell, sh.N, RI, nsz, lapse, ka, et,
                       ks, temp, amp, oka, oet, oks, otemp, oamp);
    return hipGetLastError();
}

// ---------------------------------------------------------------- luminosity seed

// dL_N/dpsi for L_N = c A_{I+1/2} sum_k W_k H_{I+1/2,k} with free streaming H = psi of the
// last zone: c R_{I+1/2}^2 W_k in the outermost zone (R^2 / a^2 with a lapse), zero elsewhere
// (and zero everywhere when there is no outgoing flux).
__global__ __launch_bounds__(kBlock) void k_lum_seed(Shape sh, const double* __restrict__ r_edge,
                                                     const double* __restrict__ lapse_edge,
                                                     const Consts* __restrict__ cs, const double* add,
                                                     double* seed) {
    const long long sys = blockIdx.x;
    const int I = sh.I, N = sh.N;
    const int ray = (int)(sys % sh.R);
    const bool flux = (sh.terms & kDiffusion) && sh.outer_bc == 1;
    const size_t eo = (size_t)ray * (I + 1) + I;
    const double ae = lapse_edge ? lapse_edge[eo] : 1.0;      // with a lapse the area is R^2 / a^2
    const double ro = r_edge[eo] / ae;
    const size_t n = (size_t)I * N;
    for (size_t j = threadIdx.x; j < n; j += kBlock) {
        const int i = (int)(j / N), k = (int)(j % N);
        const size_t c = (size_t)sys * n + j;
        const double a = add ? add[c] : 0.0;
        seed[c] = ((flux && i == I - 1) ? kCLight * ro * ro * cs->W[k] : 0.0) + a;
    }
}

hipError_t launch_lum_seed(const Shape& sh, const double* r_edge, const double* lapse_edge, const Consts* cs,
                           const double* add, double* seed, hipStream_t st) {
    const long long nsys = (long long)sh.S * sh.R;
    hipLaunchKernelGGL(k_lum_seed, dim3((unsigned)nsys), dim3(kBlock), 0, st, sh, r_edge, lapse_edge, cs, add, seed);
    return hipGetLastError();
}

// ---------------------------------------------------------------- line-search backtrack

__global__ __launch_bounds__(kBlock) void k_backtrack(Shape sh, double* __restrict__ psi, const double* __restrict__ dx,
                                                      int* backtrack, double* alpha) {
    const long long sys = blockIdx.x;
    if (backtrack[sys] == 0) return;
    const double a = alpha[sys];
    const double coef = 0.5 * a - a;
    const size_t n = (size_t)sh.I * sh.N;
    for (size_t j = threadIdx.x; j < n; j += kBlock) {
        const size_t cix = (size_t)sys * n + j;
        psi[cix] = psi[cix] + __dmul_rn(coef, dx[cix]);      // trial moved back to alpha / 2
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        alpha[sys] = 0.5 * a;
        backtrack[sys] = 0;
    }
}

hipError_t launch_backtrack(const Shape& sh, double* psi, const double* dx, int* backtrack, double* alpha,
                            hipStream_t st) {
    const long long nsys = (long long)sh.S * sh.R;
    hipLaunchKernelGGL(k_backtrack, dim3((unsigned)nsys), dim3(kBlock), 0, st, sh, psi, dx, backtrack, alpha);
    return hipGetLastError();
}

// ---------------------------------------------------------------- fill (a kernel rather than a memset node)

__global__ __launch_bounds__(kBlock) void k_fill_i32(int* __restrict__ p, long long n, int v) {
    const long long j = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (j < n) p[j] = v;
}

hipError_t launch_fill_i32(int* p, long long n, int v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, p, n, v);
    return hipGetLastError();
}

// ---------------------------------------------------------------- active-system count

// max |v| over each system's cells (one block per system)
__global__ __launch_bounds__(kBlock) void k_sys_absmax(const double* __restrict__ v, long long per_sys,
                                                       double* __restrict__ out) {
    __shared__ double red[kBlock / 64];
    const double* p = v + (size_t)blockIdx.x * per_sys;
    double m = 0.0;
    for (long long c = threadIdx.x; c < per_sys; c += kBlock) m = fmax(m, fabs(p[c]));
    m = block_max(m, red);
    if (threadIdx.x == 0) out[blockIdx.x] = m;
}

hipError_t launch_sys_absmax(const double* v, long long nsys, long long per_sys, double* out, hipStream_t st) {
    if (nsys <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_sys_absmax, dim3((unsigned)nsys), dim3(kBlock), 0, st, v, per_sys, out);
    return hipGetLastError();
}

// Final per-system flags of a Newton step from the last evaluated (accepted) residual: keeps the
// factorisation's zero-pivot / fallback bits, sets 1 when rtol > 0 and max|G| is above its target,
// 2 when the residual is not finite.
// One block; also the per-system statistics the caller asked for, and all flags together in *any (host memory).
__global__ __launch_bounds__(1024) void k_finish(long long n, const double* __restrict__ res, const double* __restrict__ res0,
                                                 const double* __restrict__ tgt, double rtol, const int* __restrict__ iters,
                                                 int* __restrict__ flags, double* res_out, double* res0_out, int* iters_out,
                                                 int* flags_out, int* any) {
    __shared__ int s_any;
    if (threadIdx.x == 0) s_any = 0;
    __syncthreads();
    int all = 0;
    for (long long s = threadIdx.x; s < n; s += 1024) {
        const double r = res[s];
        int fl = flags[s] & (4 | 8);
        if (!isfinite(r)) fl |= 2;
        else if (rtol > 0.0 && !(r <= tgt[s])) fl |= 1;
        flags[s] = fl;
        all |= fl;
        if (res_out) res_out[s] = r;
        if (res0_out) res0_out[s] = res0[s];
        if (iters_out) iters_out[s] = iters[s];
        if (flags_out) flags_out[s] = fl;
    }
    atomicOr(&s_any, all);
    __syncthreads();
    if (threadIdx.x == 0) *any = s_any;
}

hipError_t launch_finish(long long n, const double* res, const double* res0, const double* tgt, double rtol,
                         const int* iters, int* flags, double* res_out, double* res0_out, int* iters_out, int* flags_out,
                         int* any, hipStream_t st) {
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(1024), 0, st, n, res, res0, tgt, rtol, iters, flags, res_out, res0_out,
                       iters_out, flags_out, any);
    return hipGetLastError();
}

// The per-system state of a Newton step at its start.
__global__ __launch_bounds__(kBlock) void k_begin(long long n, int* iters, int* flags, int* pending, int* backtrack,
                                                  int* guard) {
    const long long s = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (s < n) iters[s] = flags[s] = pending[s] = backtrack[s] = guard[s] = 0;
}

hipError_t launch_begin(long long n, int* iters, int* flags, int* pending, int* backtrack, int* guard, hipStream_t st) {
    hipLaunchKernelGGL(k_begin, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, n, iters, flags, pending,
                       backtrack, guard);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_count(const int* __restrict__ active, long long n, int* count) {
    __shared__ double red[kBlock / 64];
    double s = 0.0;
    for (long long j = threadIdx.x; j < n; j += kBlock) s += active[j];
    s = block_sum(s, red);
    if (threadIdx.x == 0) *count = (int)s;
}

// What the host decides by after a residual pass, in one launch: the active systems in ascending order, and in `out`
// (host memory) how many they are, how many trials were rejected and how many systems tripped the growth guard since
// the last call (the marks are cleared).  One block: each wavefront counts its stretch, then writes the indices
// behind those of the stretches before it.
__global__ __launch_bounds__(1024) void k_tally(const int* __restrict__ active, const int* __restrict__ backtrack,
                                                int* __restrict__ guard, long long n, int* __restrict__ list, int* out) {
    __shared__ int s_n[16][3];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long len = ((n + 1023) / 1024) * 64, lo = wave * len, hi = min(n, lo + len);
    int mine[3] = {0, 0, 0};
    for (long long j = lo + lane; j < hi; j += 64) {
        const int g = guard[j];
        mine[0] += active[j] != 0;
        mine[1] += backtrack[j] != 0;
        mine[2] += g != 0;
        if (g) guard[j] = 0;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mine[k] += __shfl_xor(mine[k], o);
        if (lane == 0) s_n[wave][k] = mine[k];
    }
    __syncthreads();
    int at = 0;
    for (int w = 0; w < wave; ++w) at += s_n[w][0];
    for (long long j0 = lo; j0 < hi; j0 += 64) {
        const long long j = j0 + lane;
        const bool on = j < hi && active[j] != 0;
        const unsigned long long m = __ballot(on);
        if (on) list[at + __popcll(m & ((1ull << lane) - 1))] = (int)j;
        at += __popcll(m);
    }
    if (threadIdx.x < 3) {
        int sum = 0;
        for (int w = 0; w < 16; ++w) sum += s_n[w][threadIdx.x];
        out[threadIdx.x] = sum;
    }
}

hipError_t launch_tally(const int* active, const int* backtrack, int* guard, long long n, int* list, int* out,
                        hipStream_t st) {
    hipLaunchKernelGGL(k_tally, dim3(1), dim3(1024), 0, st, active, backtrack, guard, n, list, out);
    return hipGetLastError();
}

hipError_t launch_count_active(const int* active, long long n, int* count, hipStream_t st) {
    hipLaunchKernelGGL(k_count, dim3(1), dim3(kBlock), 0, st, active, n, count);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_mark(const int* __restrict__ guard, long long n, int* __restrict__ act,
                                                 int* count) {
    __shared__ double red[kBlock / 64];
    double s = 0.0;
    for (long long j = threadIdx.x; j < n; j += kBlock) {
        const int v = guard[j] != 0;
        act[j] = v;
        s += v;
    }
    s = block_sum(s, red);
    if (threadIdx.x == 0) *count = (int)s;
}

__global__ __launch_bounds__(kBlock) void k_count_bits(const int* __restrict__ flags, long long n, int mask,
                                                       int* count) {
    __shared__ double red[kBlock / 64];
    double s = 0.0;
    for (long long j = threadIdx.x; j < n; j += kBlock) s += (flags[j] & mask) != 0;
    s = block_sum(s, red);
    if (threadIdx.x == 0) *count = (int)s;
}

hipError_t launch_count_bits(const int* flags, long long n, int mask, int* count, hipStream_t st) {
    hipLaunchKernelGGL(k_count_bits, dim3(1), dim3(kBlock), 0, st, flags, n, mask, count);
    return hipGetLastError();
}

hipError_t launch_mark(const int* guard, long long n, int* active_out, int* count, hipStream_t st) {
    hipLaunchKernelGGL(k_mark, dim3(1), dim3(kBlock), 0, st, guard, n, active_out, count);
    return hipGetLastError();
}

// ---------------------------------------------------------------- dispatch on the padded group count

int padded_groups(int N) {
    static const int sizes[] = {4, 8, 12, 16, 20, 24, 28, 32};
    for (int s : sizes)
        if (N <= s) return s;
    return -1;
}

#define TM_DISPATCH_NT(NTV, ...)                                       \
    switch (NTV) {                                                     \
        case 4: { constexpr int NT = 4; __VA_ARGS__; } break;          \
        case 8: { constexpr int NT = 8; __VA_ARGS__; } break;          \
        case 12: { constexpr int NT = 12; __VA_ARGS__; } break;        \
        case 16: { constexpr int NT = 16; __VA_ARGS__; } break;        \
        case 20: { constexpr int NT = 20; __VA_ARGS__; } break;        \
        case 24: { constexpr int NT = 24; __VA_ARGS__; } break;        \
        case 28: { constexpr int NT = 28; __VA_ARGS__; } break;        \
        case 32: { constexpr int NT = 32; __VA_ARGS__; } break;        \
        default: return hipErrorInvalidValue;                          \
    }

hipError_t launch_residual(const Shape& sh, const Fields& f, const Consts* cs, const double* psi_n,
                           const double* psi, double* G_out, double g_sign, const ResidualOut& out,
                           hipStream_t st) {
    const long long nsys = (long long)sh.S * sh.R;
    const bool geo = sh.limiter == 2 || sh.outer_bc == 2;
    const int groups = padded_groups(sh.N);
    if (groups < 0) return hipErrorInvalidValue;
    // Threads by cells or sixteen-zone chunks.  Up to four groups the cells, except that the geometric options (more
    // registers and arithmetic a cell) gain by the chunks once the chip is full: 768 systems of 100 zones x 4 groups 25
    // against 28 us, 1024: 30 against 28.5, 32768: 0.37 against 0.34 ms.  With more groups the chunks, but for rays so
    // short that one wavefront works alone through the groups of a few zones, while a block of cells has them all at
    // once: few systems (256 of 10 zones x 32 groups 28.5 against 33 us, of 4 x 24 22 against 27; 1024 of 15 x 32 43
    // against 38), and a ray that is one chunk of rows up to 1024 systems (1024 of 4 zones x 20 groups 25 against 28 us,
    // 8192: 73 against 68) or of more than 24 groups (8192 of 4 x 28 89 against 108, of 4 x 24 79 against 77).
    const bool one_chunk = sh.I <= kBlock / groups - 2;
    const bool by_cells = sh.N <= 4 ? !(geo && nsys > 768)
                                    : (one_chunk && (nsys <= 1024 || sh.N > 24)) || (sh.I <= 15 && nsys <= 512);
    if (by_cells) {
        const dim3 grid((unsigned)nsys), block(kBlock);
        if (geo) {
            TM_DISPATCH_NT(groups, hipLaunchKernelGGL((k_residual_rows<NT, true, true>), grid, block, 0, st, sh, f, cs, psi_n,
                                                   psi, G_out, g_sign, out));
        } else if (f.lapse) {
            TM_DISPATCH_NT(groups, hipLaunchKernelGGL((k_residual_rows<NT, true, false>), grid, block, 0, st, sh, f, cs, psi_n,
                                                   psi, G_out, g_sign, out));
        } else {
            TM_DISPATCH_NT(groups, hipLaunchKernelGGL((k_residual_rows<NT, false, false>), grid, block, 0, st, sh, f, cs, psi_n,
                                                   psi, G_out, g_sign, out));
        }
        return hipGetLastError();
    }
    // The fewest wavefronts that take no more chunks each than four would: one without zones holds registers and LDS for
    // nothing.  Against four wavefronts with a quarter of the ray each, 40000 systems: of 4 zones x 8 groups 0.29 -> 0.091
    // ms, 4 x 20 0.64 -> 0.23, 30 x 20 0.76 -> 0.60, 40 x 20 0.80 -> 0.64, 60 x 20 1.19 -> 0.95.
    auto each = [&](int W) { return (sh.I + W - 1 + 15 * W - 1) / (15 * W); };
    auto chunks = [&](auto waves) -> hipError_t {
        constexpr int W = decltype(waves)::value;
        const dim3 grid((unsigned)nsys), block(64 * W);
        if (geo) {
            TM_DISPATCH_NT(groups, hipLaunchKernelGGL((k_residual<NT / 4, true, W>), grid, block, 0, st, sh, f, cs,
                                                                   psi_n, psi, G_out, g_sign, out));
        } else {
            TM_DISPATCH_NT(groups, hipLaunchKernelGGL((k_residual<NT / 4, false, W>), grid, block, 0, st, sh, f,
                                                                   cs, psi_n, psi, G_out, g_sign, out));
        }
        return hipGetLastError();
    };
    if (each(1) == each(4)) return chunks(std::integral_constant<int, 1>());
    if (each(2) == each(4)) return chunks(std::integral_constant<int, 2>());
    if (each(3) == each(4)) return chunks(std::integral_constant<int, 3>());
    return chunks(std::integral_constant<int, 4>());
}

hipError_t launch_blocks(const Shape& sh, const Fields& f, const Consts* cs, const double* psi, double* blocks,
                         hipStream_t st) {
    const long long nsys = (long long)sh.S * sh.R;
    TM_DISPATCH_NT(padded_groups(sh.N),
                   hipLaunchKernelGGL(k_blocks<NT>, dim3((unsigned)nsys), dim3(kBlock), 0, st, sh, f, cs, psi,
                                      blocks));
    return hipGetLastError();
}

hipError_t launch_vjp(const Shape& sh, const Fields& f, const Consts* cs, const double* psi, const double* mu,
                      double* g_ka, double* g_eta, double* g_ks, double* g_amp, hipStream_t st) {
    const long long nsys = (long long)sh.S * sh.R;
    TM_DISPATCH_NT(padded_groups(sh.N),
                   hipLaunchKernelGGL(k_vjp<NT>, dim3((unsigned)nsys), dim3(kBlock), 0, st, sh, f, cs, psi, mu,
                                      g_ka, g_eta, g_ks, g_amp));
    return hipGetLastError();
}

}  // namespace tmk

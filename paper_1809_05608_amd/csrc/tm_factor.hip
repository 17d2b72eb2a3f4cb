// Lane kernels of the block-Thomas factor/solve (bodies in tm_factor_body.hpp): the instantiations without
// the geometric options, and the dispatch of every factor launch (the quad kernel, the tile and wave kernels, these, or
// the geometric instantiations of tm_factor_geo.hip).
#include "tm_factor_body.hpp"

namespace tmk {

size_t factor_ws_bytes_per_system(int I, int N, bool fp32) {
    const int NT = padded_groups(N);
    if (NT < 0) return 0;
    const size_t es = fp32 ? 4 : 8;
    return (size_t)I * NT * (NT + 1) * es;
}

// Up to this many systems, three workgroups to each of 256 CUs, what counts is the time of one wavefront's step: half
// a system per pair of wavefronts (tm_factor_w.hip) is the faster, above it four half systems per wavefront
// (tm_factor_t.hip), whose matrix operations have no idle rows.  Measured, 540 zones x 20 groups: 6 systems 0.93
// against 1.90 ms, 24: 1.00 against 2.00, 512: 1.35 against 2.00, 720: 1.65 against 2.16, 1024: 2.35 against 2.23,
// 1536: 3.1 against 2.3.  The line is that of 20 groups for all: at others the two cross later, so a little above it
// (300 zones, 1024 systems) the tiles are the slower by 7% at 8 groups (0.44 against 0.47), 5% at 12 (0.60 against
// 0.63) and 14% at 28 (2.1 against 2.4).  The count is that of all batches: a batch takes the kernel that the whole
// would take.
constexpr long long kWaveSystems = 768;

// Up to four groups a block is one tile, and the tile kernel's wavefront carries two systems where lanes by rows
// carry four: above this many systems, where all SIMDs are busy, the lanes are the faster.  Tiles against lanes, 300
// zones x 4 groups: 8192 systems 0.75 against 1.25 ms, 16384: 1.33 against 1.36, 32768: 2.40 against 1.91; one group,
// 32768 systems: 2.06 against 1.50.
constexpr long long kLaneSystems = 16384;

// As many of five to eight groups take the lanes on rays of few zones, where what the tile kernel does once per system
// is not spread over a chain: tiles against lanes, 8 groups: 32768 systems of 2 zones 0.175 against 0.146 ms, 300000 of 4
// 1.70 against 1.49, of 8 2.11 against 1.95, of 16 2.99 against 2.90 and transposed 3.09 against 3.18.  The forward
// solve up to twice the zones with the lapse and four times with the geometric options, which cost the lanes less:
// 300000 of 16 with the lapse 3.75 against 3.37, of 24 geometric 4.5 against 4.0, of 32 5.5 against 5.0; but 32768 of
// 24 with the lapse 0.61 against 0.62, 78125 of 48 geometric 2.07 against 2.03.
static bool takes_lanes(const FactorArgs& a, bool transpose) {
    if (a.list || a.total <= kLaneSystems || a.sh.N > 8) return false;
    if (a.sh.N <= 4) return true;
    const bool geo = a.sh.limiter == 2 || a.sh.outer_bc == 2;
    return a.sh.I <= (transpose ? 8 : geo ? 32 : a.f.lapse ? 16 : 8);
}

// Up to this many systems a float32 launch leaves the chip waiting for one wavefront's chain of zones, 16 systems
// from one end: the FP64 kernels with two or half a system per wavefront from both ends are faster up to about
// twice as many, float32 the faster above for half the bytes of factors.  float32 against FP64, 540 zones x 20
// groups: 720 systems 7.0 against 2.2 ms, 4096: 7.1 against 4.0, 8192: 8.1 against 7.7, 16384: 10.9 against 15.1;
// 300 zones, 4096 systems: 8 groups 1.12 against 0.65, 12: 1.79 against 1.11, 16: 2.74 against 1.63, 24: 4.87
// against 4.18, 32: 7.64 against 7.03.
constexpr long long kFp64Systems = 4096;

static bool near_cells(const Shape& sh) { return (long long)sh.S * sh.R * sh.I * sh.N < (1ll << 29); }

bool factor_takes_list(const Shape& sh, long long systems) {
    return systems <= kWaveSystems || near_cells(sh);       // the tile kernel reaches a pair's cells with 32-bit offsets
}

// A workspace of float32 size holds half as many FP64 systems.  Two launches that each wait for the chain then cost
// more than the one of float32, except where that is slowest (one wavefront's quads, 5 to 20 groups) and where the
// wavefront per half ray is the quickest: a step of 4 updates, 300 zones, float32 against two launches of FP64: 4096
// systems x 24 groups 18.4 against 21.0 ms, 32: 28.4 against 33.9, 2048 x 32: 20.3 against 21.3; 4096 x 20: 14.9
// against 11.5, 4096 x 8: 4.4 against 4.1; 100 zones, 768 systems of 4 groups 0.85 against 0.74, 4096: 1.03
// against 1.16.
bool factor_in_fp64(const Shape& sh, long long systems, long long slots) {
    return systems <= kFp64Systems && (systems == (long long)sh.S * sh.R || factor_takes_list(sh, systems)) &&
           (systems <= slots || systems <= kWaveSystems || (sh.N > 4 && sh.N <= 20));
}

long long factor_fp64_slots(const Shape& sh, size_t bytes) {
    return (long long)(bytes / factor_ws_bytes_per_system(sh.I, sh.N, false)) & ~1ll;     // whole pairs
}

hipError_t launch_factor(const FactorArgs& a, bool fp32, bool transpose, bool pivot, hipStream_t st, int kernel) {
    // the float32 forward solve with diagonal pivots (the mixed-precision Newton update) takes one
    // system per quad of lanes up to 20 groups
    if (kernel != kFactorLane && fp32 && !transpose && !pivot &&
        launch_factor_quad(a, st, kernel))
        return hipGetLastError();
    // FP64 with diagonal pivots: on the matrix cores, both ends of a ray at once, for every option and, but for very
    // many systems of few groups (takes_lanes), every group count (one row per lane: 8.2 ms against 2.1 at 720 systems of
    // 540 zones x 20 groups, 122 against 58 at 65536; five groups of 100 zones, 65536 systems: 2.92 against 2.63).  The
    // tile kernel addresses the cells of two systems with 32-bit byte offsets.
    if (!fp32 && !pivot) {
        const bool few = a.total <= kWaveSystems, far = (long long)a.sh.I * a.sh.N >= (1ll << 27);
        if (!takes_lanes(a, transpose)) return few || far ? launch_factor_wave(a, transpose, st) : launch_factor_tile(a, transpose, st);
    }
    if (a.sh.limiter == 2 || a.sh.outer_bc == 2) return launch_factor_geo(a, fp32, transpose, pivot, st);
    return launch_lane<false>(a, fp32, transpose, pivot, st);
}

}  // namespace tmk

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

// Up to this many systems the two wavefronts of each have a SIMD to themselves (256 CUs of four), and what
// counts is the time of one wavefront's step: half a system per wavefront (tm_factor_w.hip) is the faster, above
// it four half systems per wavefront (tm_factor_t.hip), whose matrix operations have no idle rows.  Measured,
// 540 zones x 20 groups: 6 systems 1.28 against 1.90 ms, 24: 1.45 against 2.00, 512: 1.99 against 2.00, 1024:
// 2.20 against 2.23, 2048: 4.6 against 2.6; 300 x 12: 1024 systems 0.65 against 0.63, 2048 1.10 against 0.76.
// The count is the problem's, not the launch's: a batch takes the kernel that the whole would take.
constexpr long long kWaveSystems = 512;

hipError_t launch_factor(const FactorArgs& a, bool fp32, bool transpose, bool pivot, hipStream_t st, int kernel) {
    // the float32 forward solve with diagonal pivots (the mixed-precision Newton update) takes one
    // system per quad of lanes up to 20 groups
    if (kernel != kFactorLane && fp32 && !transpose && !pivot &&
        launch_factor_quad(a, st, kernel))
        return hipGetLastError();
    // FP64 with diagonal pivots: on the matrix cores, both ends of a ray at once, for every group count and
    // option (one row per lane: 8.2 ms against 2.1 at 720 systems, 122 against 57 at 65536).  The tile kernel
    // addresses the cells of two systems with 32-bit byte offsets.
    if (!fp32 && !pivot) {
        const bool few = (long long)a.sh.S * a.sh.R <= kWaveSystems, far = (long long)a.sh.I * a.sh.N >= (1ll << 27);
        return few || far ? launch_factor_wave(a, transpose, st) : launch_factor_tile(a, transpose, st);
    }
    if (a.sh.limiter == 2 || a.sh.outer_bc == 2) return launch_factor_geo(a, fp32, transpose, pivot, st);
    return launch_lane<false>(a, fp32, transpose, pivot, st);
}

}  // namespace tmk

// Lane kernels of the block-Thomas factor/solve (bodies in tm_factor_body.hpp): the instantiations without
// the geometric options, and the dispatch of every factor launch (the quad kernel, the tile kernel, these, or
// the geometric instantiations of tm_factor_geo.hip).
#include "tm_factor_body.hpp"

namespace tmk {

size_t factor_ws_bytes_per_system(int I, int N, bool fp32) {
    const int NT = padded_groups(N);
    if (NT < 0) return 0;
    const size_t es = fp32 ? 4 : 8;
    return (size_t)I * NT * (NT + 1) * es;
}

hipError_t launch_factor(const FactorArgs& a, bool fp32, bool transpose, bool pivot, hipStream_t st, int kernel) {
    // the float32 forward solve with diagonal pivots (the mixed-precision Newton update) takes one
    // system per quad of lanes up to 20 groups
    if (kernel != kFactorLane && fp32 && !transpose && !pivot &&
        launch_factor_quad(a, st, kernel))
        return hipGetLastError();
    // FP64 with diagonal pivots: matrix-core tiles, both ends of a ray at once, for every group count and
    // option (one row per lane: 8.2 ms against 2.1 at 720 systems, 122 against 58.7 at 65536).  The tile
    // kernel addresses the cells of two systems with 32-bit byte offsets; a ray beyond that takes the
    // partial-pivoting kernel.
    if (!fp32 && !pivot) {
        if ((long long)a.sh.I * a.sh.N < (1ll << 27)) return launch_factor_tile(a, transpose, st);
        pivot = true;
    }
    if (a.sh.limiter == 2 || a.sh.outer_bc == 2) return launch_factor_geo(a, fp32, transpose, pivot, st);
    return launch_lane<false>(a, fp32, transpose, pivot, st);
}

}  // namespace tmk

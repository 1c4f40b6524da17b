// The relaxed flows' two-launch passes in float, and the precision dispatch.
#include "mbo_fastrelax_launch.hpp"

namespace mbo {

hipError_t launch_row_fast_relax_f64(int n, int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare);
hipError_t launch_resolvent_fast_f64(int log2L, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare);

hipError_t launch_row_fast_relax(int prec, int n, int log2L, const FastRowArgs& a, dim3 grid, hipStream_t st,
                                 bool prepare)
{
    if (prec == 1) return row_fast_relax_t<float>(n, log2L, a, grid, st, prepare);
    return launch_row_fast_relax_f64(n, log2L, a, grid, st, prepare);
}

hipError_t launch_resolvent_fast(int prec, int log2L, const FastColArgs& a, dim3 grid, hipStream_t st, bool prepare)
{
    if (prec == 1) return resolvent_fast_t<float>(log2L, a, grid, st, prepare);
    return launch_resolvent_fast_f64(log2L, a, grid, st, prepare);
}

int resolvent_fast_tile(int log2L) { return resolvent_tile(log2L); }

}  // namespace mbo

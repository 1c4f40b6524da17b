// The relaxed flows' two-launch passes in double.
#include "mbo_fastrelax_launch.hpp"

namespace mbo {

hipError_t launch_row_fast_relax_f64(int n, int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    return row_fast_relax_t<double>(n, log2L, a, g, st, prepare);
}

hipError_t launch_resolvent_fast_f64(int log2L, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    return resolvent_fast_t<double>(log2L, a, g, st, prepare);
}

}  // namespace mbo

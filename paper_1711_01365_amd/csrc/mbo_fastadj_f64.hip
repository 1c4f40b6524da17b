// The adjoint step's band-limited passes in double (the row pass for n = 2).
#include "mbo_fastadj_launch.hpp"

namespace mbo {

hipError_t launch_row_fast_vjp_f64(int n, int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    if (n == 2) return row_fast_vjp_n<double, 2>(log2L, a, g, st, prepare);
    return hipErrorInvalidValue;
}

hipError_t launch_heat_fast_adj_f64(int log2L, int mode, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    return heat_fast_adj_t<double>(log2L, mode, a, g, st, prepare);
}

}  // namespace mbo

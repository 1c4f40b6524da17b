// The adjoint step's band-limited passes in float, and the precision dispatch.
#include "mbo_fastadj_launch.hpp"

namespace mbo {

hipError_t launch_row_fast_vjp_f64(int n, int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare);
hipError_t launch_heat_fast_adj_f64(int log2L, int mode, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare);

// n = 2, and n = 3 in float: the instances whose registers hold the product
// beside the row pass (4 x 4 and double 3 x 3 Jacobi would spill).
bool row_fast_vjp_served(int prec, int n) { return n == 2 || (n == 3 && prec == 1); }

hipError_t launch_row_fast_vjp(int prec, int n, int log2L, const FastRowArgs& a, dim3 grid, hipStream_t st,
                               bool prepare)
{
    if (prec != 1) return launch_row_fast_vjp_f64(n, log2L, a, grid, st, prepare);
    if (n == 2) return row_fast_vjp_n<float, 2>(log2L, a, grid, st, prepare);
    if (n == 3) return row_fast_vjp_n<float, 3>(log2L, a, grid, st, prepare);
    return hipErrorInvalidValue;
}

hipError_t launch_heat_fast_adj(int prec, int log2L, int mode, const FastColArgs& a, dim3 grid, hipStream_t st,
                                bool prepare)
{
    if (prec == 1) return heat_fast_adj_t<float>(log2L, mode, a, grid, st, prepare);
    return launch_heat_fast_adj_f64(log2L, mode, a, grid, st, prepare);
}

int heat_fast_adj_tile(int log2L) { return adj_tile(log2L); }

}  // namespace mbo

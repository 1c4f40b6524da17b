// The volume-preserving step's band-limited passes in float, and the precision
// dispatch.
#include "mbo_fastvol_launch.hpp"

namespace mbo {

hipError_t launch_row_fast_vkey_f64(int n, int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare);
hipError_t launch_volume_fix_f64(int n, const VolFixArgs& a, dim3 g, hipStream_t st);
hipError_t launch_volume_redo_f64(int n, int log2L, const VolFixArgs& a, dim3 g, hipStream_t st, bool prepare);

hipError_t launch_row_fast_vkey(int prec, int n, int log2L, const FastRowArgs& a, dim3 grid, hipStream_t st,
                                bool prepare)
{
    if (prec == 1) return row_fast_vkey_t<float>(n, log2L, a, grid, st, prepare);
    return launch_row_fast_vkey_f64(n, log2L, a, grid, st, prepare);
}

hipError_t launch_volume_fix(int prec, int n, const VolFixArgs& a, dim3 grid, hipStream_t st)
{
    if (prec == 1) return volume_fix_t<float>(n, a, grid, st);
    return launch_volume_fix_f64(n, a, grid, st);
}

hipError_t launch_volume_redo(int prec, int n, int log2L, const VolFixArgs& a, dim3 grid, hipStream_t st, bool prepare)
{
    if (prec == 1) return volume_redo_t<float>(n, log2L, a, grid, st, prepare);
    return launch_volume_redo_f64(n, log2L, a, grid, st, prepare);
}

}  // namespace mbo

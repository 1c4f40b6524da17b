// The volume-preserving step's band-limited passes in double.
#include "mbo_fastvol_launch.hpp"

namespace mbo {

hipError_t launch_row_fast_vkey_f64(int n, int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    return row_fast_vkey_t<double>(n, log2L, a, g, st, prepare);
}

hipError_t launch_volume_fix_f64(int n, const VolFixArgs& a, dim3 g, hipStream_t st)
{
    return volume_fix_t<double>(n, a, g, st);
}

hipError_t launch_volume_redo_f64(int n, int log2L, const VolFixArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    return volume_redo_t<double>(n, log2L, a, g, st, prepare);
}

}  // namespace mbo

// 3-D plane pass in float, and the precision dispatch of its launcher.
#include "mbo_plane_launch.hpp"

namespace mbo {

hipError_t launch_plane_fast_f64(int log2Y, int log2Z, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare,
                                 hipEvent_t ev0, hipEvent_t ev1);

hipError_t launch_plane_fast(int prec, int log2Y, int log2Z, const FastColArgs& a, dim3 grid, hipStream_t st,
                             bool prepare, hipEvent_t ev0, hipEvent_t ev1)
{
    if (prec == 1) return plane_fast_t<float>(log2Y, log2Z, a, grid, st, prepare, ev0, ev1);
    return launch_plane_fast_f64(log2Y, log2Z, a, grid, st, prepare, ev0, ev1);
}

int plane_fast_group(int log2Y, int log2Z)
{
    const int threads = (1 << (log2Y + log2Z)) / 16;
    return threads < 64 ? 64 / threads : 1;
}

int plane_fast_threads(int log2Y, int log2Z)
{
    return plane_fast_group(log2Y, log2Z) * ((1 << (log2Y + log2Z)) / 16);
}

size_t plane_fast_lds_bytes(int prec, int log2Y, int log2Z)
{
    const size_t ny = (size_t)1 << log2Y, nz = (size_t)1 << log2Z;
    return ((size_t)plane_fast_group(log2Y, log2Z) * nz * (ny + 1) + ny + nz) * 2 *
           (prec == 1 ? sizeof(float) : sizeof(double));
}

}  // namespace mbo

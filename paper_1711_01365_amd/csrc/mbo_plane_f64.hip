// 3-D plane pass in double.
#include "mbo_plane_launch.hpp"

namespace mbo {

hipError_t launch_plane_fast_f64(int log2Y, int log2Z, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare,
                                 hipEvent_t ev0, hipEvent_t ev1)
{
    return plane_fast_t<double>(log2Y, log2Z, a, g, st, prepare, ev0, ev1);
}

}  // namespace mbo

// Launcher of the 3-D plane pass (plane_fast, mbo_fast.hpp) for one precision T:
// sides of 8 to 128 points in double and of 64 or 128 in float whose plane fits the LDS.
#pragma once

#include <hip/hip_ext.h>

#include "mbo_fast.hpp"

namespace mbo {

constexpr size_t PLANE_LDS_MAX = 160 * 1024;

template <typename T, int LY, int LZ>
static hipError_t plane_fast_go(const FastColArgs& a, dim3 g, hipStream_t st, bool prepare, hipEvent_t ev0,
                                hipEvent_t ev1)
{
    typedef PlaneFastShape<T, LY, LZ> S;
    if constexpr (S::LDS > PLANE_LDS_MAX || (sizeof(T) == 4 && (LY < 6 || LZ < 6))) {
        return hipErrorInvalidValue;
    } else {
        const void* f = reinterpret_cast<const void*>(&plane_fast<T, LY, LZ>);
        if (prepare) return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
        if (ev0) hipExtLaunchKernelGGL((plane_fast<T, LY, LZ>), g, dim3(S::THREADS), S::LDS, st, ev0, ev1, 0, a);
        else hipLaunchKernelGGL((plane_fast<T, LY, LZ>), g, dim3(S::THREADS), S::LDS, st, a);
        return hipGetLastError();
    }
}

template <typename T, int LY>
static hipError_t plane_fast_y(int log2Z, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare,
                               hipEvent_t ev0, hipEvent_t ev1)
{
    switch (log2Z) {
    case 3: return plane_fast_go<T, LY, 3>(a, g, st, prepare, ev0, ev1);
    case 4: return plane_fast_go<T, LY, 4>(a, g, st, prepare, ev0, ev1);
    case 5: return plane_fast_go<T, LY, 5>(a, g, st, prepare, ev0, ev1);
    case 6: return plane_fast_go<T, LY, 6>(a, g, st, prepare, ev0, ev1);
    case 7: return plane_fast_go<T, LY, 7>(a, g, st, prepare, ev0, ev1);
    }
    return hipErrorInvalidValue;
}

template <typename T>
static hipError_t plane_fast_t(int log2Y, int log2Z, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare,
                               hipEvent_t ev0, hipEvent_t ev1)
{
    switch (log2Y) {
    case 3: return plane_fast_y<T, 3>(log2Z, a, g, st, prepare, ev0, ev1);
    case 4: return plane_fast_y<T, 4>(log2Z, a, g, st, prepare, ev0, ev1);
    case 5: return plane_fast_y<T, 5>(log2Z, a, g, st, prepare, ev0, ev1);
    case 6: return plane_fast_y<T, 6>(log2Z, a, g, st, prepare, ev0, ev1);
    case 7: return plane_fast_y<T, 7>(log2Z, a, g, st, prepare, ev0, ev1);
    }
    return hipErrorInvalidValue;
}

}  // namespace mbo

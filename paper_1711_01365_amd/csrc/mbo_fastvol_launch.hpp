// Launchers of the volume-preserving step's band-limited passes (row_fast_vkey,
// volume_fix and volume_redo, mbo_fast.hpp) for one precision T.
#pragma once

#include "mbo_fast.hpp"

namespace mbo {

template <typename T, int n, int LG>
static hipError_t row_fast_vkey_go(const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    typedef RowFastShape<T, n, LG> S;
    if constexpr (S::LDS > 163840) {
        return hipErrorInvalidValue;  // no plan has this shape (its lines do not fit in LDS)
    } else {
        const void* f = reinterpret_cast<const void*>(&row_fast_vkey<T, n, LG>);
        if (prepare) return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
        hipLaunchKernelGGL((row_fast_vkey<T, n, LG>), g, dim3(S::THREADS), S::LDS, st, a);
        return hipGetLastError();
    }
}

template <typename T, int n>
static hipError_t row_fast_vkey_n(int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    return with_row_length(log2L, [&](auto lg) { return row_fast_vkey_go<T, n, lg.value>(a, g, st, prepare); });
}

template <typename T>
static hipError_t row_fast_vkey_t(int n, int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    switch (n) {
    case 1: return row_fast_vkey_n<T, 1>(log2L, a, g, st, prepare);
    case 2: return row_fast_vkey_n<T, 2>(log2L, a, g, st, prepare);
    case 3: return row_fast_vkey_n<T, 3>(log2L, a, g, st, prepare);
    case 4: return row_fast_vkey_n<T, 4>(log2L, a, g, st, prepare);
    }
    return hipErrorInvalidValue;
}

template <typename T, int n, int LG>
static hipError_t volume_redo_go(const VolFixArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    typedef RowFastShape<T, n, LG> S;
    if constexpr (S::LDS > 163840) {
        return hipErrorInvalidValue;  // no plan has this shape (its lines do not fit in LDS)
    } else {
        const void* f = reinterpret_cast<const void*>(&volume_redo<T, n, LG>);
        if (prepare) return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
        hipLaunchKernelGGL((volume_redo<T, n, LG>), g, dim3(S::THREADS), S::LDS, st, a);
        return hipGetLastError();
    }
}

template <typename T, int n>
static hipError_t volume_redo_n(int log2L, const VolFixArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    return with_row_length(log2L, [&](auto lg) { return volume_redo_go<T, n, lg.value>(a, g, st, prepare); });
}

template <typename T>
static hipError_t volume_redo_t(int n, int log2L, const VolFixArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    switch (n) {
    case 1: return volume_redo_n<T, 1>(log2L, a, g, st, prepare);
    case 2: return volume_redo_n<T, 2>(log2L, a, g, st, prepare);
    case 3: return volume_redo_n<T, 3>(log2L, a, g, st, prepare);
    case 4: return volume_redo_n<T, 4>(log2L, a, g, st, prepare);
    }
    return hipErrorInvalidValue;
}

template <typename T, int n>
static hipError_t volume_fix_n(const VolFixArgs& a, dim3 g, hipStream_t st)
{
    const size_t lds = (size_t)a.r.L * 2 * sizeof(T);  // at most 32 KiB
    hipLaunchKernelGGL((volume_fix<T, n>), g, dim3(VFIX_NT), lds, st, a);
    return hipGetLastError();
}

template <typename T>
static hipError_t volume_fix_t(int n, const VolFixArgs& a, dim3 g, hipStream_t st)
{
    switch (n) {
    case 1: return volume_fix_n<T, 1>(a, g, st);
    case 2: return volume_fix_n<T, 2>(a, g, st);
    case 3: return volume_fix_n<T, 3>(a, g, st);
    case 4: return volume_fix_n<T, 4>(a, g, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace mbo

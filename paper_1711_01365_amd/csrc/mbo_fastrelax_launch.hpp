// Launchers of the relaxed flows' passes (row_fast_relax and the column pass in mode
// HF_RESOLVENT, mbo_fast.hpp) for one precision T.
#pragma once

#include "mbo_fast.hpp"

namespace mbo {

template <typename T, int n, int LG>
static hipError_t row_fast_relax_go(const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    typedef RowFastShape<T, n, LG> S;
    if constexpr (S::LDS > 163840) {
        return hipErrorInvalidValue;  // no plan has this shape (its lines do not fit in LDS)
    } else {
        const void* f = reinterpret_cast<const void*>(&row_fast_relax<T, n, LG>);
        if (prepare) return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
        hipLaunchKernelGGL((row_fast_relax<T, n, LG>), g, dim3(S::THREADS), S::LDS, st, a);
        return hipGetLastError();
    }
}

template <typename T, int n>
static hipError_t row_fast_relax_n(int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    return with_row_length(log2L, [&](auto lg) { return row_fast_relax_go<T, n, lg.value>(a, g, st, prepare); });
}

template <typename T>
static hipError_t row_fast_relax_t(int n, int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    switch (n) {
    case 1: return row_fast_relax_n<T, 1>(log2L, a, g, st, prepare);
    case 2: return row_fast_relax_n<T, 2>(log2L, a, g, st, prepare);
    case 3: return row_fast_relax_n<T, 3>(log2L, a, g, st, prepare);
    }
    return hipErrorInvalidValue;
}

// Columns per workgroup: four (32-byte segments of a float row), two for 2048 rows
// (more would not fit 256 registers in double), more where four would leave less
// than one wave.  512 x 512, n = 3 in float: 14.7 us with 2, 12.3 with 4, 12.8
// with 8; in double 17.6, 16.4, 20.8; 1024 x 512 in float 25.2 and 22.3.
constexpr int resolvent_tile(int log2L) { return log2L >= 11 ? 2 : log2L >= 8 ? 4 : 512 >> log2L; }

template <typename T, int LG>
static hipError_t resolvent_fast_go(const FastColArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    constexpr int TX = resolvent_tile(LG), NT = TX * (1 << LG) / 8;
    const size_t lds = HeatFastShape<T, LG, TX>::LDS;
    const void* f = reinterpret_cast<const void*>(&heat_fast_adj<T, LG, TX, HF_RESOLVENT>);
    if (prepare) return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((heat_fast_adj<T, LG, TX, HF_RESOLVENT>), g, dim3(NT), lds, st, a);
    return hipGetLastError();
}

template <typename T>
static hipError_t resolvent_fast_t(int log2L, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    switch (log2L) {
    case 6: return resolvent_fast_go<T, 6>(a, g, st, prepare);
    case 7: return resolvent_fast_go<T, 7>(a, g, st, prepare);
    case 8: return resolvent_fast_go<T, 8>(a, g, st, prepare);
    case 9: return resolvent_fast_go<T, 9>(a, g, st, prepare);
    case 10: return resolvent_fast_go<T, 10>(a, g, st, prepare);
    case 11: return resolvent_fast_go<T, 11>(a, g, st, prepare);
    }
    return hipErrorInvalidValue;
}

}  // namespace mbo

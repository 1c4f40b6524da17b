// Launchers of the adjoint step's band-limited passes (row_fast_vjp and
// heat_fast_adj, mbo_fast.hpp) for one precision T.
#pragma once

#include "mbo_fast.hpp"

namespace mbo {

template <typename T, int n, int LG>
static hipError_t row_fast_vjp_go(const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    typedef RowFastShape<T, n, LG> S;
    if constexpr (S::LDS > 163840) {
        return hipErrorInvalidValue;  // no plan has this shape (its lines do not fit in LDS)
    } else {
        const void* f = reinterpret_cast<const void*>(&row_fast_vjp<T, n, LG>);
        if (prepare) return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
        hipLaunchKernelGGL((row_fast_vjp<T, n, LG>), g, dim3(S::THREADS), S::LDS, st, a);
        return hipGetLastError();
    }
}

template <typename T, int n>
static hipError_t row_fast_vjp_n(int log2L, const FastRowArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    return with_row_length(log2L, [&](auto lg) { return row_fast_vjp_go<T, n, lg.value>(a, g, st, prepare); });
}

// Columns per workgroup of heat_fast_adj: two, more where that would leave
// less than one wave (the default rule of the plain pass).
constexpr int adj_tile(int log2L) { return log2L >= 8 ? 2 : 512 >> log2L; }

template <typename T, int LG>
static hipError_t heat_fast_adj_go(int mode, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    constexpr int TX = adj_tile(LG), NT = TX * (1 << LG) / 8;
    const size_t lds = HeatFastShape<T, LG, TX>::LDS;
    if (prepare) {
        const void* fs[3] = {reinterpret_cast<const void*>(&heat_fast_adj<T, LG, TX, HF_SAVE>),
                             reinterpret_cast<const void*>(&heat_fast_adj<T, LG, TX, HF_DOT>),
                             reinterpret_cast<const void*>(&heat_fast_adj<T, LG, TX, HF_DTAU>)};
        for (const void* f : fs) {
            const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    if (mode == HF_SAVE) hipLaunchKernelGGL((heat_fast_adj<T, LG, TX, HF_SAVE>), g, dim3(NT), lds, st, a);
    else if (mode == HF_DOT) hipLaunchKernelGGL((heat_fast_adj<T, LG, TX, HF_DOT>), g, dim3(NT), lds, st, a);
    else if (mode == HF_DTAU) hipLaunchKernelGGL((heat_fast_adj<T, LG, TX, HF_DTAU>), g, dim3(NT), lds, st, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <typename T>
static hipError_t heat_fast_adj_t(int log2L, int mode, const FastColArgs& a, dim3 g, hipStream_t st, bool prepare)
{
    switch (log2L) {
    case 6: return heat_fast_adj_go<T, 6>(mode, a, g, st, prepare);
    case 7: return heat_fast_adj_go<T, 7>(mode, a, g, st, prepare);
    case 8: return heat_fast_adj_go<T, 8>(mode, a, g, st, prepare);
    case 9: return heat_fast_adj_go<T, 9>(mode, a, g, st, prepare);
    case 10: return heat_fast_adj_go<T, 10>(mode, a, g, st, prepare);
    case 11: return heat_fast_adj_go<T, 11>(mode, a, g, st, prepare);
    }
    return hipErrorInvalidValue;
}

}  // namespace mbo

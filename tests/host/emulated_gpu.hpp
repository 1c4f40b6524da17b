// Kernels on the CPU: included in front of a kernel source, it makes the source plain C++
// whose launches run each workgroup as fibers on one thread (emulated_gpu.cpp), so that an
// address sanitizer sees every access.  64 lanes of a wave meet at shuffles and ballots,
// the workgroup at __syncthreads; workgroups run one after another, launches at once.
// __shared__ variables become static, so that a declaration of dynamic shared memory
// (extern __shared__) has to be taken out of the text before.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <functional>

#undef hipLaunchKernelGGL
#undef __global__
#undef __device__
#undef __shared__
#undef __forceinline__
#undef __launch_bounds__
#undef __HIP_MEMORY_SCOPE_AGENT
#undef __HIP_MEMORY_SCOPE_WORKGROUP
#define __global__
#define __device__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __HIP_MEMORY_SCOPE_AGENT 4
#define __HIP_MEMORY_SCOPE_WORKGROUP 3

namespace emulated {
struct Lane {
    dim3 tid;
    int lane, wave;
};
const Lane& self();
extern dim3 block, block_dim, grid_dim;
extern unsigned long long exchange[16 * 64], votes[16];  // per wave of the workgroup
void wg_sync();
void wave_sync(int site);  // the lanes of a wave that wait at one site go on together
void run(dim3 grid, dim3 block, const std::function<void()>& kernel);

template <typename T>
T shuffle(T v, int from, int site)
{
    static_assert(sizeof(T) <= 8, "a word");
    unsigned long long* x = exchange + self().wave * 64;
    std::memcpy(x + self().lane, &v, sizeof v);
    wave_sync(site);
    std::memcpy(&v, x + (from & 63), sizeof v);
    wave_sync(site + 1);
    return v;
}
unsigned long long ballot(bool p, int site);

template <typename T, typename U, typename F>
T update(T* p, U v, F f)
{
    const T old = *p;
    *p = f(old, (T)v);
    return old;
}
}  // namespace emulated

#define threadIdx (emulated::self().tid)
#define blockIdx emulated::block
#define blockDim emulated::block_dim
#define gridDim emulated::grid_dim
#define __syncthreads() emulated::wg_sync()
#define __threadfence() ((void)0)
#define EMULATED_SITE (__LINE__ * 4)
#define __shfl_xor(v, m, w) emulated::shuffle((v), emulated::self().lane ^ (int)(m), EMULATED_SITE)
#define __shfl_up(v, d, w)                                                                                  \
    emulated::shuffle((v), emulated::self().lane >= (int)(d) ? emulated::self().lane - (int)(d)             \
                                                             : emulated::self().lane,                       \
                      EMULATED_SITE)
#define __shfl(v, s, ...) emulated::shuffle((v), (int)(s), EMULATED_SITE)
#define __ballot(p) emulated::ballot((p), EMULATED_SITE)
#define __popcll(x) __builtin_popcountll(x)
#define __clzll(x) ((x) ? __builtin_clzll((unsigned long long)(x)) : 64)
#define __clz(x) ((x) ? __builtin_clz((unsigned)(x)) : 32)
#define __hip_atomic_load(p, o, s) (*(p))
#define __hip_atomic_exchange(p, v, o, s) emulated::update((p), (v), [](auto, auto b) { return b; })
#define __hip_atomic_fetch_add(p, v, o, s) atomicAdd((p), (v))
#define __hip_atomic_fetch_max(p, v, o, s) atomicMax((p), (v))
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsqf(x) (1.0f / sqrtf(x))
#define __builtin_amdgcn_rsq(x) (1.0 / sqrt(x))
#define __builtin_amdgcn_sqrtf(x) sqrtf(x)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_s_setprio(x) ((void)0)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() emulated::wave_sync(EMULATED_SITE)
#define hipGetLastError() hipSuccess
#define hipFuncSetAttribute(...) hipSuccess
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
    emulated::run((grid), (block), [=] { kernel(__VA_ARGS__); })

inline unsigned __float_as_uint(float v)
{
    unsigned u;
    std::memcpy(&u, &v, sizeof u);
    return u;
}
inline long long __double_as_longlong(double v)
{
    long long u;
    std::memcpy(&u, &v, sizeof u);
    return u;
}
inline double __longlong_as_double(long long u)
{
    double v;
    std::memcpy(&v, &u, sizeof v);
    return v;
}
template <typename T, typename U>
T atomicAdd(T* p, U v) { return emulated::update(p, v, [](T a, T b) { return a + b; }); }
template <typename T, typename U>
T atomicMin(T* p, U v) { return emulated::update(p, v, [](T a, T b) { return b < a ? b : a; }); }
template <typename T, typename U>
T atomicMax(T* p, U v) { return emulated::update(p, v, [](T a, T b) { return a < b ? b : a; }); }
template <typename T, typename U>
T atomicAnd(T* p, U v) { return emulated::update(p, v, [](T a, T b) { return a & b; }); }
template <typename T, typename U>
T atomicOr(T* p, U v) { return emulated::update(p, v, [](T a, T b) { return a | b; }); }

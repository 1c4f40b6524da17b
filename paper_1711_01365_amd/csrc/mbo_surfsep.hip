// Spreading and interpolation of the surface diffusion step through the structure
// of the band (mbo_surface.hip holds the general kernels and the gridding kernel
// psi).
//
// Spreading.  The samples of all band cells are points of one tensor lattice:
// p Chebyshev nodes per lattice cell and axis, the same for every cell, with
// weights that factor per axis.  The spread grid is therefore a product of three
// one-dimensional maps applied to the lattice values (zero outside the band),
//     G[x][y][z] = sum_i Wx[x][i] sum_j Wy[y][j] sum_k Wz[z][k] v[i][j][k],
// each banded (a grid point sees the nodes within w / 2 of it): three passes that
// move the values a few times instead of forming each cell's block of U^3 grid
// points.  The weights of a pass are a table, [node of the run][grid point], built
// once in double.  Unit sphere with dx = 0.05, p = 3 (3.3 M samples, 128^3 grid),
// n = 3 in float: 92 + 109 + 124 us for the z, y and x passes, which move 253, 244
// and 194 MB (2.8, 2.2 and 1.6 TB/s; bound by the loads of a workgroup's lines and
// then by the products from LDS, one after the other).  The cell contraction with
// its tile gather took 2060 + 450.
//
// Interpolation.  Targets that share their stencil start (about 150 of them on the
// paper's sphere) read the same w^3 grid values: a wave takes up to 64 of them, the
// values come as scalar loads and each lane keeps its own weights.  Bound by VALU
// issue, w^3 products per target and entry (0.6 ms of the 0.93 it takes there, 1.45
// with the general kernel, whose LDS tile returns each value once per target); the
// rest is the latency of the scalar loads, which eight waves per SIMD (40
// registers) and contiguous runs of groups per XCD keep short: 1.46 ms without
// them.
#include <algorithm>

#include "mbo_kernels.hpp"

namespace mbo {

// A run's weights are padded with zeros to a multiple of this (a second run starts
// there): the unit of the scalar weight loads.
constexpr int SEP_PAD = SURF_SEP_PAD;

// ---------------------------------------------------------------------------
// z pass: one workgroup per (column of cells, group of entries)
// ---------------------------------------------------------------------------
// A column is the cells of one (i, j); its samples are contiguous.  The workgroup
// lays them out as lines of the whole lattice in LDS (zeros between the cells),
// P^2 lines for p <= 4, else the P lines of one node a.  A thread owns one grid
// point of one entry and adds up all lines of it, so that a weight is read once.
template <typename T, int P, int AB>
__global__ void __launch_bounds__(512) sep_z(const SurfSepArgs a)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int p3 = P * P * P, NA = AB == P * P ? 1 : P;  // launches of a column per entry
    T* lds = reinterpret_cast<T*>(smem_raw);
    const int Ng = a.Ng, Lz = a.len[2];
    const int E = blockDim.x / Ng;  // entries at a time
    const int tid = threadIdx.x;
    const int col = blockIdx.x;
    const int eg = blockIdx.y / NA, an = blockIdx.y - eg * NA;
    const int64_t c0 = a.col_start[col];
    const int nc = (int)(a.col_start[col + 1] - c0);
    const int lines = E * AB;
    for (int i = tid; i < lines * Lz; i += blockDim.x) lds[i] = (T)0;
    __syncthreads();
    const T* A = reinterpret_cast<const T*>(a.A);
    for (int s = 0; s < E; ++s) {
        const int e = eg * E + s;
        if (e >= a.nn) break;
        const T* src = A + (size_t)e * a.m + c0 * p3;
        if constexpr (NA == 1) {
            for (int i = tid; i < nc * p3; i += blockDim.x) {
                const int c = i / p3, r = i - c * p3, ab = r / P, ce = r - ab * P;
                lds[(s * AB + ab) * Lz + a.cell_k[c0 + c] * P + ce] = src[i];
            }
        } else {
            for (int i = tid; i < nc * P * P; i += blockDim.x) {
                const int c = i / (P * P), r = i - c * P * P, b = r / P, ce = r - b * P;
                lds[(s * AB + b) * Lz + a.cell_k[c0 + c] * P + ce] = src[c * p3 + an * P * P + r];
            }
        }
    }
    __syncthreads();
    const int s = tid / Ng, g = tid - s * Ng, e = eg * E + s;
    if (s >= E || e >= a.nn) return;
    const SepRun r = a.run[2][g];
    const T* w = reinterpret_cast<const T*>(a.w[2]) + g;  // [node of the run][grid point]
    T acc[AB];
#pragma unroll
    for (int k = 0; k < AB; ++k) acc[k] = (T)0;
    const T* v = lds + s * AB * Lz;
    for (int n = 0; n < r.len0; ++n) {
        const T wt = w[(size_t)n * Ng];
#pragma unroll
        for (int k = 0; k < AB; ++k) acc[k] += wt * v[k * Lz + r.n0 + n];
    }
    const int b1 = (r.len0 + SEP_PAD - 1) & ~(SEP_PAD - 1);
    for (int n = 0; n < r.len1; ++n) {
        const T wt = w[(size_t)(b1 + n) * Ng];
#pragma unroll
        for (int k = 0; k < AB; ++k) acc[k] += wt * v[k * Lz + r.n1 + n];
    }
    T* out = reinterpret_cast<T*>(a.t1) + (((size_t)e * a.ncols + col) * (P * P) + (NA == 1 ? 0 : an * P)) * Ng + g;
#pragma unroll
    for (int k = 0; k < AB; ++k) out[(size_t)k * Ng] = acc[k];
}

// ---------------------------------------------------------------------------
// y and x passes: lines of nodes across, two entries and ZT neighbouring z points
// at a time
// ---------------------------------------------------------------------------
// The lines of a workgroup sit in LDS, node n of entry h at ((h rows) + n - lo +
// SEP_PAD) ZT, with SEP_PAD rows of zeros on both sides.  A half (ZT = 32) or a
// part of a wave is one entry, so a wave works on one grid point g (ZT = 32; two
// or four with 16 or 8) and the weights of g come as scalar loads, SEP_PAD at a
// time: two instructions per product.

// out = sum over the runs of g, clipped to the nodes [lo, hi) in steps of SEP_PAD
// (beyond them the rows are zeros, and so are the weights past a run's end).
template <typename T, int ZT, typename WP>
__device__ __forceinline__ T sep_sum(const T* col, int lo, int hi, const SepRun& r, WP w)
{
    T s = 0;
    int n = r.n0 < lo ? (lo - r.n0) & ~(SEP_PAD - 1) : 0;
    int ne = r.n0 + r.len0 > hi ? hi - r.n0 : r.len0;
    for (; n < ne; n += SEP_PAD) {
        const T* v = col + (r.n0 + n - lo + SEP_PAD) * ZT;
#pragma unroll
        for (int k = 0; k < SEP_PAD; ++k) s += w[n + k] * v[k * ZT];
    }
    const int base = (r.len0 + SEP_PAD - 1) & ~(SEP_PAD - 1);
    n = r.n1 < lo ? (lo - r.n1) & ~(SEP_PAD - 1) : 0;
    ne = r.n1 + r.len1 > hi ? hi - r.n1 : r.len1;
    for (; n < ne; n += SEP_PAD) {
        const T* v = col + (r.n1 + n - lo + SEP_PAD) * ZT;
#pragma unroll
        for (int k = 0; k < SEP_PAD; ++k) s += w[base + n + k] * v[k * ZT];
    }
    return s;
}

// The grid points of a workgroup's lines: g runs over the waves' parts.
template <typename T, int ZT, typename Store>
__device__ __forceinline__ void sep_lines(const SurfSepArgs& a, int axis, const T* col, int lo, int hi, Store store)
{
    typedef const __attribute__((address_space(4))) T* Uniform;
    constexpr int PER = 64 / (2 * ZT);  // grid points per wave
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int Ng = a.Ng;
    if constexpr (PER == 1) {
        for (int g = wave; g < Ng; g += 4) {
            const SepRun r = a.run[axis][g];
            const Uniform w = (Uniform)(uintptr_t)a.w[axis] + (size_t)g * a.wlen[axis];
            store(g, sep_sum<T, ZT>(col, lo, hi, r, w));
        }
    } else {
        for (int g = wave * PER + ((int)threadIdx.x & 63) / (2 * ZT); g < Ng; g += 4 * PER) {
            const SepRun r = a.run[axis][g];
            const T* w = reinterpret_cast<const T*>(a.w[axis]) + (size_t)g * a.wlen[axis];
            store(g, sep_sum<T, ZT>(col, lo, hi, r, w));
        }
    }
}

// One workgroup per (x node, z tile, entry pair): the columns of the node's slice,
// every y grid point.
template <typename T, int ZT>
__global__ void __launch_bounds__(256) sep_y(const SurfSepArgs a)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* tile = reinterpret_cast<T*>(smem_raw);
    const int Ng = a.Ng, p = a.p, tid = threadIdx.x;
    const int t = blockIdx.x, i = t / p, an = t - i * p;  // node a of lattice cell i
    const int z0 = blockIdx.y * ZT;
    const int cs = a.slice[i], ce = a.slice[i + 1];
    int lo = 0, hi = 0;  // the slice's y nodes
    if (ce > cs) {
        lo = a.col_j[cs] * p;
        hi = (a.col_j[ce - 1] + 1) * p;
    }
    const int rows = hi - lo + 2 * SEP_PAD;
    const int z = tid % ZT, h = (tid / ZT) & 1, q = tid / (2 * ZT);
    constexpr int Q = 256 / (2 * ZT);
    const int e = 2 * blockIdx.z + h;
    const bool live = e < a.nn;
    if ((hi - lo) != (ce - cs) * p) {  // gaps between the columns
        for (int n = tid; n < 2 * rows * ZT; n += 256) tile[n] = (T)0;
        __syncthreads();
    }
    T* col = tile + (size_t)h * rows * ZT + z;
    for (int n = q; n < 2 * SEP_PAD; n += Q) col[(n < SEP_PAD ? n : rows - 2 * SEP_PAD + n) * ZT] = (T)0;
    const T* src = reinterpret_cast<const T*>(a.t1) + ((size_t)(live ? e : 0) * a.ncols) * (p * p) * Ng + z0 + z;
#pragma unroll 4
    for (int n = q; n < (ce - cs) * p; n += Q) {
        const int c = n / p, b = n - c * p;
        col[(a.col_j[cs + c] * p + b - lo + SEP_PAD) * ZT] = src[((size_t)(cs + c) * (p * p) + an * p + b) * Ng];
    }
    __syncthreads();
    T* out = reinterpret_cast<T*>(a.t2) + (((size_t)(live ? e : 0) * a.len[0] + t) * Ng) * Ng + z0 + z;
    sep_lines<T, ZT>(a, 1, col, lo, hi, [&](int g, T v) {
        if (live) out[(size_t)g * Ng] = v;
    });
}

// One workgroup per (y grid point, z tile, packed plane): every x grid point, the
// plane's two entries as real and imaginary part.
template <typename T, int ZT>
__global__ void __launch_bounds__(256) sep_x(const SurfSepArgs a)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* tile = reinterpret_cast<T*>(smem_raw);
    const int Ng = a.Ng, tid = threadIdx.x, Lx = a.len[0], rows = Lx + 2 * SEP_PAD;
    const int y = blockIdx.x, z0 = blockIdx.y * ZT, pl = blockIdx.z;
    const int z = tid % ZT, h = (tid / ZT) & 1, q = tid / (2 * ZT);
    constexpr int Q = 256 / (2 * ZT);
    const int e = 2 * pl + h;
    const bool live = e < a.nn;
    const size_t node = (size_t)Ng * Ng;
    T* col = tile + (size_t)h * rows * ZT + z;
    for (int n = q; n < 2 * SEP_PAD; n += Q) col[(n < SEP_PAD ? n : rows - 2 * SEP_PAD + n) * ZT] = (T)0;
    const T* src = reinterpret_cast<const T*>(a.t2) + (size_t)(live ? e : 0) * Lx * node + (size_t)y * Ng + z0 + z;
#pragma unroll 8
    for (int n = q; n < Lx; n += Q) col[(n + SEP_PAD) * ZT] = live ? src[n * node] : (T)0;
    __syncthreads();
    T* out = reinterpret_cast<T*>(a.Z) + 2 * ((size_t)pl * Ng * node + (size_t)y * Ng + z0 + z) + h;
    sep_lines<T, ZT>(a, 0, col, 0, Lx, [&](int g, T v) { out[2 * (size_t)g * node] = v; });
}

// ---------------------------------------------------------------------------
// Interpolation of targets grouped by stencil start
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T es_weight(T z, T invW, T beta)
{
    const T r = z * invW;
    const T s = (T)1 - r * r;
    if constexpr (sizeof(T) == 4) {
        const float b2 = beta * 1.4426950408889634f;  // beta log2(e)
        return s > 0.0f ? __builtin_amdgcn_exp2f(b2 * __builtin_amdgcn_sqrtf(s) - b2) : 0.0f;
    } else {
        return s > (T)0 ? exp(beta * (sqrt(s) - (T)1)) : (T)0;
    }
}

template <typename T, int W2, int n>
__global__ void __launch_bounds__(256, sizeof(T) == 4 ? 8 : 4) surface_interp_groups(const SurfArgs a, const SurfGroup* __restrict__ groups,
                                                             int ngroups)
{
    constexpr int NN = n * n, PL = (NN + 1) / 2;
    // the grid is read-only here and its addresses are the same for a whole wave
    typedef const __attribute__((address_space(4))) T* Uniform;
    // the eight XCDs (own L2 each) take contiguous runs of groups, whose stencils overlap
    const unsigned per = (gridDim.x + 7) >> 3, wg = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    const int gi = __builtin_amdgcn_readfirstlane((int)(wg * 4 + (threadIdx.x >> 6)));
    if (gi >= ngroups) return;
    const SurfGroup gr = groups[gi];
    const int lane = threadIdx.x & 63;
    const bool live = lane < gr.count;
    const int64_t s = gr.first + (live ? lane : 0);
    const T* pos = reinterpret_cast<const T*>(a.pos);
    const T beta = (T)a.beta, invh = (T)(1.0 / a.h), y0 = (T)a.y0, invW = (T)1 / ((T)W2 * (T)0.5);
    T wx[W2], wy[W2], wz[W2];
    {
        const T ux = (pos[s] - y0) * invh, uy = (pos[a.m + s] - y0) * invh, uz = (pos[2 * a.m + s] - y0) * invh;
#pragma unroll
        for (int k = 0; k < W2; ++k) {
            wx[k] = es_weight<T>((T)(gr.i0 + k) - ux, invW, beta);
            wy[k] = es_weight<T>((T)(gr.j0 + k) - uy, invW, beta);
            wz[k] = es_weight<T>((T)(gr.k0 + k) - uz, invW, beta);
        }
    }
    const int64_t q = a.perm[s];
    const int64_t Ng = a.Ng, npts = Ng * Ng * Ng;
    const Uniform Z = (Uniform)(uintptr_t)a.Z;
    T acc[2 * PL];
#pragma unroll
    for (int k = 0; k < 2 * PL; ++k) acc[k] = (T)0;
#pragma unroll 1
    for (int j = 0; j < W2; ++j) {
        // the y weight of this row, by selects (wy stays in registers)
        T wj = wy[0];
#pragma unroll
        for (int k = 1; k < W2; ++k) wj = j == k ? wy[k] : wj;
#pragma unroll
        for (int i = 0; i < W2; ++i) {
            const T wij = wx[i] * wj;
            const int64_t row = ((gr.i0 + i) * Ng + (gr.j0 + j)) * Ng + gr.k0;
#pragma unroll
            for (int pl = 0; pl < PL; ++pl) {
                const Uniform v = Z + 2 * (pl * npts + row);
                T zr = 0, zi = 0;
#pragma unroll
                for (int k = 0; k < W2; ++k) {
                    zr += wz[k] * v[2 * k];
                    if (2 * pl + 1 < NN) zi += wz[k] * v[2 * k + 1];
                }
                acc[2 * pl] += wij * zr;
                if (2 * pl + 1 < NN) acc[2 * pl + 1] += wij * zi;
            }
        }
    }
    if (!live) return;
    T* out = reinterpret_cast<T*>(a.out);
#pragma unroll
    for (int k = 0; k < NN; ++k) out[(size_t)k * a.m + q] = acc[k];
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
template <typename T, int P>
static hipError_t sep_z_p(const SurfSepArgs& a, hipStream_t st, size_t prepare_lds)
{
    constexpr int AB = P <= 4 ? P * P : P;
    const int nt = a.Ng > 256 ? a.Ng : 256, E = nt / a.Ng;
    const size_t lds = (size_t)E * AB * a.len[2] * sizeof(T);
    if (prepare_lds)
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&sep_z<T, P, AB>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)prepare_lds);
    const dim3 g((unsigned)a.ncols, (unsigned)(((a.nn + E - 1) / E) * (AB == P * P ? 1 : P)));
    hipLaunchKernelGGL((sep_z<T, P, AB>), g, dim3(nt), lds, st, a);
    return hipGetLastError();
}

template <typename T, int ZT>
static hipError_t sep_yx(const SurfSepArgs& a, hipStream_t st, size_t prepare_lds)
{
    const size_t ly = (size_t)2 * (a.len[1] + 2 * SEP_PAD) * ZT * sizeof(T);
    const size_t lx = (size_t)2 * (a.len[0] + 2 * SEP_PAD) * ZT * sizeof(T);
    if (prepare_lds) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sep_y<T, ZT>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)prepare_lds);
        if (e != hipSuccess) return e;
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&sep_x<T, ZT>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)prepare_lds);
    }
    const unsigned zt = (unsigned)(a.Ng / ZT);
    hipLaunchKernelGGL((sep_y<T, ZT>), dim3((unsigned)a.len[0], zt, (unsigned)((a.nn + 1) / 2)), dim3(256), ly, st,
                       a);
    hipLaunchKernelGGL((sep_x<T, ZT>), dim3((unsigned)a.Ng, zt, (unsigned)((a.nn + 1) / 2)), dim3(256), lx, st, a);
    return hipGetLastError();
}

// LDS bytes of the largest workgroup of the three passes, and the z tile of the
// y and x passes: the widest of 32, 16, 8 points whose lines leave room for two
// workgroups per CU (the passes load and then compute), or fit at all.
int sep_tile(int len_x, int len_y, size_t esz, size_t lds_max)
{
    const size_t l = (size_t)2 * (std::max(len_x, len_y) + 2 * SEP_PAD) * esz;
    for (int zt = 32; zt >= 8; zt /= 2)
        if (l * zt <= lds_max / 2) return zt;
    return l * 8 <= lds_max ? 8 : 0;
}

size_t sep_z_lds(int p, int len_z, int Ng, size_t esz)
{
    const int nt = Ng > 256 ? Ng : 256;
    return (size_t)(nt / Ng) * (p <= 4 ? p * p : p) * len_z * esz;
}

template <typename T>
static hipError_t sep_t(const SurfSepArgs& a, hipStream_t st, size_t prepare_lds)
{
    if (a.Ng < 64 || a.Ng > 512 || a.Ng % 32 || a.ncols < 1) return hipErrorInvalidValue;
    hipError_t e = hipErrorInvalidValue;
    switch (a.p) {
    case 1: e = sep_z_p<T, 1>(a, st, prepare_lds); break;
    case 2: e = sep_z_p<T, 2>(a, st, prepare_lds); break;
    case 3: e = sep_z_p<T, 3>(a, st, prepare_lds); break;
    case 4: e = sep_z_p<T, 4>(a, st, prepare_lds); break;
    case 5: e = sep_z_p<T, 5>(a, st, prepare_lds); break;
    case 6: e = sep_z_p<T, 6>(a, st, prepare_lds); break;
    case 7: e = sep_z_p<T, 7>(a, st, prepare_lds); break;
    case 8: e = sep_z_p<T, 8>(a, st, prepare_lds); break;
    }
    if (e != hipSuccess) return e;
    switch (a.zt) {
    case 32: return sep_yx<T, 32>(a, st, prepare_lds);
    case 16: return sep_yx<T, 16>(a, st, prepare_lds);
    case 8: return sep_yx<T, 8>(a, st, prepare_lds);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_surface_sep(int prec, const SurfSepArgs& a, hipStream_t st, size_t prepare_lds)
{
    return prec == 0 ? sep_t<double>(a, st, prepare_lds) : sep_t<float>(a, st, prepare_lds);
}

template <typename T, int W2>
static hipError_t interp_w(const SurfArgs& a, const SurfGroup* gr, int ng, hipStream_t st)
{
    const dim3 g((unsigned)((ng + 31) / 32 * 8)), bl(256);  // a multiple of the XCDs
    switch (a.n) {
    case 1: hipLaunchKernelGGL((surface_interp_groups<T, W2, 1>), g, bl, 0, st, a, gr, ng); break;
    case 2: hipLaunchKernelGGL((surface_interp_groups<T, W2, 2>), g, bl, 0, st, a, gr, ng); break;
    case 3: hipLaunchKernelGGL((surface_interp_groups<T, W2, 3>), g, bl, 0, st, a, gr, ng); break;
    case 4: hipLaunchKernelGGL((surface_interp_groups<T, W2, 4>), g, bl, 0, st, a, gr, ng); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T>
static hipError_t interp_t(const SurfArgs& a, const SurfGroup* gr, int ng, hipStream_t st)
{
    switch (a.w) {
    case 3: return interp_w<T, 3>(a, gr, ng, st);
    case 4: return interp_w<T, 4>(a, gr, ng, st);
    case 5: return interp_w<T, 5>(a, gr, ng, st);
    case 6: return interp_w<T, 6>(a, gr, ng, st);
    case 7: return interp_w<T, 7>(a, gr, ng, st);
    case 8: return interp_w<T, 8>(a, gr, ng, st);
    case 9: return interp_w<T, 9>(a, gr, ng, st);
    case 10: return interp_w<T, 10>(a, gr, ng, st);
    case 11: return interp_w<T, 11>(a, gr, ng, st);
    case 12: return interp_w<T, 12>(a, gr, ng, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_surface_interp_groups(int prec, const SurfArgs& a, const SurfGroup* groups, int ngroups,
                                        hipStream_t st)
{
    if (ngroups <= 0) return hipSuccess;
    return prec == 0 ? interp_t<double>(a, groups, ngroups, st) : interp_t<float>(a, groups, ngroups, st);
}

}  // namespace mbo

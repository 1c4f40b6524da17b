// Selection kernels of the volume-preserving step (Section 7 of Osting & Wang,
// arXiv:1711.01365): per field, the n_plus points with the largest Delta E
// (the flat-torus rule of choosing the first n_plus values in descending
// order), equal values taken in ascending point index.
//
// Radix search over order-preserving keys of Delta E (vp_key), SEL_BITS bits
// per pass from the top: a pass histograms the next digit of the keys that
// match the digits found so far (one workgroup per chunk of SEL_CHUNK points,
// LDS histogram, non-zero bins added to the field's global
// histogram), and one workgroup per field then finds the digit holding the
// n_plus-th largest key and clears the histogram.  After the last digit the
// key kstar is known; when only some of the points with key kstar are
// selected, per-chunk counts of those points and a walk through the chunk
// holding the last selected one give its index istar (sel_tie).  Every kernel
// reads the selection state first and returns at once when its field needs no
// more work.
#include <climits>

#include "mbo_kernels.hpp"

namespace mbo {

// Inclusive scan over a 256-thread workgroup (four waves); total receives the
// sum over the workgroup.  Every thread must call it.
__device__ __forceinline__ long long scan256(long long v, long long* sh /* >= 4 */, long long& total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    if (lane == 63) sh[w] = v;
    __syncthreads();
    long long add = 0;
    for (int i = 0; i < w; ++i) add += sh[i];
    total = sh[0] + sh[1] + sh[2] + sh[3];
    __syncthreads();  // sh is free for the next call
    return v + add;
}

template <typename T>
__global__ void __launch_bounds__(256) sel_hist(const SelArgs a, int shift, int bits, int pass)
{
    constexpr int KB = (int)sizeof(T) * 8;
    __shared__ unsigned h[1 << SEL_BITS];
    const int b = blockIdx.y;
    const long long np = a.nplus[b];
    if (np <= 0 || np >= a.npts) return;  // decided without a search
    if (pass > 0 && a.st[b].mode != VS_SEARCH) return;
    const int top = shift + bits;
    const unsigned long long pre = pass > 0 ? a.st[b].kstar : 0ull;
    const int nb = 1 << bits;
    for (int i = threadIdx.x; i < nb; i += blockDim.x) h[i] = 0u;
    __syncthreads();
    const T* v = reinterpret_cast<const T*>(a.dE) + (size_t)b * a.npts;
    const int64_t x0 = (int64_t)blockIdx.x * SEL_CHUNK + threadIdx.x;
    T val[SEL_PER];
#pragma unroll
    for (int k = 0; k < SEL_PER; ++k) {  // every load in flight at once
        const int64_t x = x0 + (int64_t)k * 256;
        val[k] = x < a.npts ? v[x] : (T)0;
    }
    // equal digits that follow each other in a thread count once (smooth fields:
    // most points of a chunk share the digit, and the lanes' atomics on its bin
    // are done one after another)
    unsigned bin = 0u, run = 0u;
#pragma unroll
    for (int k = 0; k < SEL_PER; ++k) {
        const unsigned long long key = vp_key(val[k]);
        if (x0 + (int64_t)k * 256 < a.npts && (top >= KB || (key >> top) == (pre >> top))) {
            const unsigned d = (unsigned)(key >> shift) & (unsigned)(nb - 1);
            if (run && d != bin) {
                atomicAdd(&h[bin], run);
                run = 0u;
            }
            bin = d;
            ++run;
        }
    }
    if (run) atomicAdd(&h[bin], run);
    __syncthreads();
    unsigned* g = a.hist + (size_t)b * (1 << SEL_BITS);
    for (int i = threadIdx.x; i < nb; i += blockDim.x)
        if (h[i]) atomicAdd(&g[i], h[i]);
}

__global__ void __launch_bounds__(256) sel_pick(const SelArgs a, int shift, int bits, int pass, int last)
{
    __shared__ long long sh[4];
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    VpSel* st = a.st + b;
    const long long np = a.nplus[b];
    if (pass == 0) {
        if (np <= 0 || np >= a.npts) {
            if (tid == 0) {
                st->mode = np <= 0 ? VS_NONE : VS_ALL;
                st->kstar = 0ull;
                st->need = 0;
                st->ties = 0;
                st->istar = -1;
            }
            return;
        }
    } else if (st->mode != VS_SEARCH) {
        return;
    }
    const long long need = pass == 0 ? np : st->need;
    const unsigned long long pre = pass == 0 ? 0ull : st->kstar;
    unsigned* g = a.hist + (size_t)b * (1 << SEL_BITS);
    const int nb = 1 << bits;
    const int per = nb >> 8;  // bins per thread (bits >= 9)
    // thread t holds the t-th group of bins from the top, in descending order
    const int hi = nb - 1 - tid * per;
    unsigned c[8];
    long long sum = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        c[i] = i < per ? g[hi - i] : 0u;
        sum += c[i];
    }
    long long total;
    const long long incl = scan256(sum, sh, total);
    const long long excl = incl - sum;
    if (excl < need && need <= incl) {  // exactly one thread
        long long acc = excl;
        int d = hi;
        unsigned cnt = c[0];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < per && acc + (long long)c[i] >= need) {
                d = hi - i;
                cnt = c[i];
                break;
            }
            acc += c[i];
        }
        const long long rem = need - acc;
        st->kstar = pre | ((unsigned long long)d << shift);
        st->need = rem;
        st->ties = cnt;
        st->mode = VS_SEARCH;
        if (last) {
            st->mode = rem == (long long)cnt ? VS_TIES_ALL : VS_TIES_PART;
            st->istar = rem == (long long)cnt ? LLONG_MAX : -1;
        }
    }
    __syncthreads();  // every bin has been read
    for (int i = tid; i < nb; i += 256) g[i] = 0u;
}

// Points whose key is kstar, per chunk; the workgroup of a field that finishes
// last then finds the chunk holding the need-th of them (in index order) and
// walks it for that point's index.  The per-chunk counts and the finished-
// workgroup counter are only touched by device-scope atomics, performed at the
// device's coherence point for workgroups on every XCD: a workgroup's count is
// performed once its returned value is in (before the barrier that precedes
// the counter), and the last workgroup's atomic reads come after the counter
// told it every other workgroup had counted; no cache write-back is needed.
template <typename T>
__global__ void __launch_bounds__(256) sel_tie(const SelArgs a)
{
    __shared__ long long sh[4];
    __shared__ long long s_chunk, s_rank;
    __shared__ int s_last;
    const int b = blockIdx.y;
    const int tid = threadIdx.x;
    VpSel* st = a.st + b;
    if (st->mode != VS_TIES_PART) return;
    const unsigned long long ks = st->kstar;
    const T* v = reinterpret_cast<const T*>(a.dE) + (size_t)b * a.npts;
    unsigned* tc = a.tcnt + (size_t)b * a.chunks;
    {
        const int64_t x0 = (int64_t)blockIdx.x * SEL_CHUNK + tid;
        T val[SEL_PER];
#pragma unroll
        for (int k = 0; k < SEL_PER; ++k) {
            const int64_t x = x0 + (int64_t)k * 256;
            val[k] = x < a.npts ? v[x] : (T)0;
        }
        long long cnt = 0;
#pragma unroll
        for (int k = 0; k < SEL_PER; ++k) cnt += (x0 + (int64_t)k * 256 < a.npts && vp_key(val[k]) == ks) ? 1 : 0;
        long long total;
        (void)scan256(cnt, sh, total);
        unsigned seen = 0u;
        if (tid == 0) seen = __hip_atomic_exchange(&tc[blockIdx.x], (unsigned)total, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
        if (seen == 0xffffffffu) s_last = 2;  // consumes the returned value (overwritten below)
        __syncthreads();
        if (tid == 0)
            s_last = __hip_atomic_fetch_add(a.done + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                             gridDim.x - 1
                         ? 1
                         : 0;
        __syncthreads();
        if (s_last != 1) return;  // uniform
        if (tid == 0) (void)__hip_atomic_exchange(a.done + b, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the last workgroup: the chunk holding the need-th tie ...
    const long long need = st->need;
    const int64_t per = (a.chunks + 255) / 256;
    const int64_t c0 = (int64_t)tid * per;
    const int64_t c1 = c0 + per < a.chunks ? c0 + per : a.chunks;
    long long sum = 0;
    for (int64_t c = c0; c < c1; ++c)
        sum += __hip_atomic_load(&tc[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid == 0) {
        s_chunk = -1;
        s_rank = 0;
    }
    long long total;
    const long long incl = scan256(sum, sh, total);  // its barriers order the writes above
    const long long excl = incl - sum;
    if (excl < need && need <= incl) {
        long long acc = excl;
        for (int64_t c = c0; c < c1; ++c) {
            const long long k = __hip_atomic_load(&tc[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (acc + k >= need) {
                s_chunk = c;
                s_rank = need - acc;
                break;
            }
            acc += k;
        }
    }
    __syncthreads();
    const long long chunk = s_chunk, rank = s_rank;
    if (chunk < 0) return;  // uniform
    // ... and the point: walk the chunk in index order
    const int64_t x0 = chunk * SEL_CHUNK;
    const int64_t x1 = x0 + SEL_CHUNK < a.npts ? x0 + SEL_CHUNK : a.npts;
    long long run = 0;
    for (int64_t xb = x0; xb < x1; xb += 256) {
        const int64_t x = xb + tid;
        const long long eq = (x < x1 && vp_key(v[x]) == ks) ? 1 : 0;
        long long tot;
        const long long r = scan256(eq, sh, tot);
        if (eq && run + r == rank) st->istar = x;
        run += tot;
        if (run >= rank) break;  // uniform: tot is the same on every thread
    }
}

// ---------------------------------------------------------------------------
// The three-launch selection (SelListArgs)
// ---------------------------------------------------------------------------

// The digit holding the cut, found by every workgroup for itself from the
// histogram (8 KB; one launch fewer than a pick kernel), then the chunk's points
// of that digit appended to the field's list, in no particular order.
template <typename T>
__global__ void __launch_bounds__(256) sel_list(const SelListArgs la, int shift)
{
    const SelArgs& a = la.s;
    __shared__ long long sh[4];
    __shared__ long long s_need;
    __shared__ int s_digit;
    __shared__ unsigned s_cnt, s_base;
    const int b = blockIdx.y, tid = threadIdx.x;
    const long long np = a.nplus[b];
    VpSel* st = a.st + b;
    if (np <= 0 || np >= a.npts) {  // uniform
        if (blockIdx.x == 0 && tid == 0) {
            st->mode = np <= 0 ? VS_NONE : VS_ALL;
            st->kstar = 0ull;
            st->need = 0;
            st->ties = 0;
            st->istar = -1;
        }
        return;
    }
    // every load of the chunk in flight while the histogram is scanned
    const T* v = reinterpret_cast<const T*>(a.dE) + (size_t)b * a.npts;
    const int64_t x0 = (int64_t)blockIdx.x * SEL_CHUNK + tid;
    T val[SEL_PER];
#pragma unroll
    for (int k = 0; k < SEL_PER; ++k) {
        const int64_t x = x0 + (int64_t)k * 256;
        val[k] = x < a.npts ? v[x] : (T)0;
    }
    const unsigned* g = a.hist + (size_t)b * (1 << SEL_BITS);
    constexpr int per = (1 << SEL_BITS) / 256;
    const int hi = (1 << SEL_BITS) - 1 - tid * per;
    unsigned c[per];
    long long sum = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
        c[i] = g[hi - i];
        sum += c[i];
    }
    if (tid == 0) s_cnt = 0u;
    long long total;
    const long long incl = scan256(sum, sh, total);
    const long long excl = incl - sum;
    if (excl < np && np <= incl) {  // exactly one thread
        long long acc = excl;
        int d = hi;
#pragma unroll
        for (int i = 0; i < per; ++i) {
            if (acc + (long long)c[i] >= np) {
                d = hi - i;
                break;
            }
            acc += c[i];
        }
        s_digit = d;
        s_need = np - acc;
    }
    __syncthreads();
    const unsigned long long digit = (unsigned long long)s_digit;
    if (blockIdx.x == 0 && tid == 0) {
        st->kstar = digit << shift;
        st->need = s_need;
        st->mode = VS_SEARCH;
        st->istar = -1;
    }
    unsigned mine = 0;
#pragma unroll
    for (int k = 0; k < SEL_PER; ++k)
        mine += (x0 + (int64_t)k * 256 < a.npts && (vp_key(val[k]) >> shift) == digit) ? 1u : 0u;
    unsigned at = mine ? atomicAdd(&s_cnt, mine) : 0u;
    __syncthreads();
    if (s_cnt == 0u) return;  // uniform
    if (tid == 0) s_base = atomicAdd(la.count + b, s_cnt);
    __syncthreads();
    at += s_base;
    unsigned long long* lk = la.key + (size_t)b * a.npts;
    unsigned* li = la.idx + (size_t)b * a.npts;
#pragma unroll
    for (int k = 0; k < SEL_PER; ++k) {
        const int64_t x = x0 + (int64_t)k * 256;
        const unsigned long long key = vp_key(val[k]);
        if (x < a.npts && (key >> shift) == digit) {
            lk[at] = key;
            li[at] = (unsigned)x;
            ++at;
        }
    }
}

// The end of the search among the listed points, one workgroup per field:
// digits of SEL_BITS bits of the key below the first, then, when only some of
// the points with the last key are selected, of the index from the lower end.
// The list is copied to LDS when it fits.  Leaves the histogram and the count at
// zero.
constexpr int SEL_LIST_LDS = 8192;
__global__ void __launch_bounds__(256) sel_finish(const SelListArgs la, int shift0, int index_bits)
{
    const SelArgs& a = la.s;
    __shared__ long long sh[4];
    __shared__ unsigned h[1 << SEL_BITS];
    __shared__ unsigned long long lkey[SEL_LIST_LDS];
    __shared__ unsigned lidx[SEL_LIST_LDS];
    __shared__ unsigned long long s_pre;
    __shared__ long long s_need;
    __shared__ unsigned s_cnt;
    const int b = blockIdx.x, tid = threadIdx.x;
    VpSel* st = a.st + b;
    const long long np = a.nplus[b];
    unsigned* g = a.hist + (size_t)b * (1 << SEL_BITS);
    const unsigned M = la.count[b];
    for (int i = tid; i < (1 << SEL_BITS); i += 256) g[i] = 0u;
    if (np <= 0 || np >= a.npts) return;  // decided by sel_list, nothing listed
    const unsigned long long* gk = la.key + (size_t)b * a.npts;
    const unsigned* gi = la.idx + (size_t)b * a.npts;
    const bool lds = M <= (unsigned)SEL_LIST_LDS;
    __syncthreads();  // every wave has read the count, which is cleared below
    if (lds)
        for (unsigned i = tid; i < M; i += 256) {
            lkey[i] = gk[i];
            lidx[i] = gi[i];
        }
    auto key_at = [&](unsigned i) { return lds ? lkey[i] : gk[i]; };
    auto idx_at = [&](unsigned i) { return lds ? lidx[i] : gi[i]; };
    if (tid == 0) {
        s_pre = st->kstar;
        s_need = st->need;
        s_cnt = M;
        la.count[b] = 0u;
    }
    __syncthreads();
    // one digit: histogram of (value >> sh) over the points for which `in`
    // holds, then the digit at which the running count, from the top (down) or
    // the bottom, reaches s_need; s_need becomes the rank within it
    auto digit = [&](auto value, auto in, int shift, int bits, bool down) -> int {
        __shared__ int s_d;
        const int nb = 1 << bits;
        for (int i = tid; i < nb; i += 256) h[i] = 0u;
        __syncthreads();
        for (unsigned i = tid; i < M; i += 256)
            if (in(i)) atomicAdd(&h[(unsigned)(value(i) >> shift) & (unsigned)(nb - 1)], 1u);
        __syncthreads();
        const int per = (nb + 255) / 256;
        long long sum = 0;
        for (int i = 0; i < per; ++i) {
            const int o = tid * per + i;
            if (o < nb) sum += h[down ? nb - 1 - o : o];
        }
        long long total;
        const long long need = s_need;
        const long long incl = scan256(sum, sh, total);
        const long long excl = incl - sum;
        if (excl < need && need <= incl) {
            long long acc = excl;
            for (int i = 0; i < per; ++i) {
                const int o = tid * per + i;
                const int d = down ? nb - 1 - o : o;
                if (acc + (long long)h[d] >= need) {
                    s_d = d;
                    s_cnt = h[d];
                    s_need = need - acc;
                    break;
                }
                acc += h[d];
            }
        }
        __syncthreads();
        return s_d;
    };
    int low = shift0;  // key bits below `low` are still open
    while (low > 0 && s_need != (long long)s_cnt) {
        const int bits = low < SEL_BITS ? low : SEL_BITS;
        const int top = low;
        low -= bits;
        const unsigned long long pre = s_pre >> top;
        const int d = digit(key_at, [&](unsigned i) { return (key_at(i) >> top) == pre; }, low, bits, true);
        if (tid == 0) s_pre |= (unsigned long long)d << low;
        __syncthreads();
    }
    const unsigned long long ks = s_pre;
    if (s_need == (long long)s_cnt) {
        // every point of the digits found is selected: the keys from ks up
        if (tid == 0) {
            st->kstar = ks;
            st->mode = VS_TIES_ALL;
            st->istar = LLONG_MAX;
        }
        return;
    }
    // the need-th smallest index among the points with key ks
    unsigned ipre = 0u;
    int ilow = index_bits;
    while (ilow > 0) {
        const int bits = ilow < SEL_BITS ? ilow : SEL_BITS;
        const int top = ilow;
        ilow -= bits;
        const unsigned pre = ipre >> top;
        const int d = digit(idx_at, [&](unsigned i) { return key_at(i) == ks && (idx_at(i) >> top) == pre; }, ilow,
                            bits, false);
        ipre |= (unsigned)d << ilow;
    }
    if (tid == 0) {
        st->kstar = ks;
        st->mode = VS_TIES_PART;
        st->istar = (long long)ipre;
    }
}

template <typename T>
__global__ void __launch_bounds__(256) sel_mark(const SelArgs a)
{
    const int b = blockIdx.y;
    const VpSel s = a.st[b];
    const T* v = reinterpret_cast<const T*>(a.dE) + (size_t)b * a.npts;
    const int64_t x0 = (int64_t)blockIdx.x * SEL_CHUNK;
    const int64_t x1 = x0 + SEL_CHUNK < a.npts ? x0 + SEL_CHUNK : a.npts;
    for (int64_t x = x0 + threadIdx.x; x < x1; x += blockDim.x)
        a.mask[(size_t)b * a.npts + x] = vp_member(s, vp_key(v[x]), x) ? 1 : 0;
}

__global__ void __launch_bounds__(256) count_pos(const int8_t* sgn, int64_t npts, long long* out)
{
    __shared__ long long sh[4];
    const int b = blockIdx.y;
    const int64_t x0 = (int64_t)blockIdx.x * SEL_CHUNK;
    const int64_t x1 = x0 + SEL_CHUNK < npts ? x0 + SEL_CHUNK : npts;
    long long cnt = 0;
    for (int64_t x = x0 + threadIdx.x; x < x1; x += blockDim.x) cnt += sgn[(size_t)b * npts + x] > 0 ? 1 : 0;
    long long total;
    (void)scan256(cnt, sh, total);
    if (threadIdx.x == 0 && total) atomicAdd(reinterpret_cast<unsigned long long*>(out + b), (unsigned long long)total);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
template <typename T>
static hipError_t select_t(const SelArgs& a, int batch, hipStream_t st)
{
    // digits from the top: float keys 11 + 11 + 10 bits, double keys 5 x 11 + 9
    static const int fs[3] = {21, 10, 0}, fb[3] = {11, 11, 10};
    static const int ds[6] = {53, 42, 31, 20, 9, 0}, db[6] = {11, 11, 11, 11, 11, 9};
    const bool f = sizeof(T) == 4;
    const int passes = f ? 3 : 6;
    const dim3 gc((unsigned)a.chunks, (unsigned)batch), gb((unsigned)batch), bl(256);
    for (int p = 0; p < passes; ++p) {
        const int sh = f ? fs[p] : ds[p], bi = f ? fb[p] : db[p];
        hipLaunchKernelGGL((sel_hist<T>), gc, bl, 0, st, a, sh, bi, p);
        hipLaunchKernelGGL(sel_pick, gb, bl, 0, st, a, sh, bi, p, p == passes - 1 ? 1 : 0);
    }
    hipLaunchKernelGGL((sel_tie<T>), gc, bl, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_select(int prec, const SelArgs& a, int batch, hipStream_t st)
{
    if (a.chunks <= 0 || batch <= 0) return hipErrorInvalidValue;
    return prec == 0 ? select_t<double>(a, batch, st) : select_t<float>(a, batch, st);
}

hipError_t launch_select_list(int prec, const SelListArgs& a, int batch, hipStream_t st)
{
    if (a.s.chunks <= 0 || batch <= 0 || a.s.npts > (1ll << 31)) return hipErrorInvalidValue;
    const dim3 gc((unsigned)a.s.chunks, (unsigned)batch), bl(256);
    const int shift = (prec == 0 ? 64 : 32) - SEL_BITS;
    int ib = 0;
    while ((1ll << ib) < a.s.npts) ++ib;
    if (prec == 0) {
        hipLaunchKernelGGL((sel_hist<double>), gc, bl, 0, st, a.s, shift, SEL_BITS, 0);
        hipLaunchKernelGGL((sel_list<double>), gc, bl, 0, st, a, shift);
    } else {
        hipLaunchKernelGGL((sel_hist<float>), gc, bl, 0, st, a.s, shift, SEL_BITS, 0);
        hipLaunchKernelGGL((sel_list<float>), gc, bl, 0, st, a, shift);
    }
    hipLaunchKernelGGL(sel_finish, dim3((unsigned)batch), bl, 0, st, a, shift, ib);
    return hipGetLastError();
}

hipError_t launch_sel_mark(int prec, const SelArgs& a, int batch, hipStream_t st)
{
    const dim3 gc((unsigned)a.chunks, (unsigned)batch), bl(256);
    if (prec == 0) hipLaunchKernelGGL((sel_mark<double>), gc, bl, 0, st, a);
    else hipLaunchKernelGGL((sel_mark<float>), gc, bl, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_count_pos(const int8_t* sgn, int64_t npts, int batch, long long* out, hipStream_t st)
{
    hipError_t e = launch_fill_u64(reinterpret_cast<unsigned long long*>(out), batch, 0ull, st);
    if (e != hipSuccess) return e;
    const dim3 gc((unsigned)((npts + SEL_CHUNK - 1) / SEL_CHUNK), (unsigned)batch), bl(256);
    hipLaunchKernelGGL(count_pos, gc, bl, 0, st, sgn, npts, out);
    return hipGetLastError();
}

hipError_t launch_row_vp(int prec, int n, int log2L, const RowArgs& a, dim3 grid, dim3 block, size_t lds,
                         hipStream_t st, bool prepare)
{
    return prec == 0 ? launch_row_vp_f64(n, log2L, a, grid, block, lds, st, prepare)
                     : launch_row_vp_f32(n, log2L, a, grid, block, lds, st, prepare);
}

}  // namespace mbo

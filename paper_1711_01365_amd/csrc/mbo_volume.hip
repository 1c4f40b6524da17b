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
#include <algorithm>
#include <climits>

#include "mbo_kernels.hpp"

namespace mbo {

// Inclusive scan over a workgroup of NT threads; total receives the sum over the
// workgroup.  Every thread must call it.
template <int NT>
__device__ __forceinline__ long long scan_wg(long long v, long long* sh /* >= NT / 64 */, long long& total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    if (lane == 63) sh[w] = v;
    __syncthreads();
    long long add = 0, all = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        const long long x = sh[i];
        add += i < w ? x : 0;
        all += x;
    }
    total = all;
    __syncthreads();  // sh is free for the next call
    return v + add;
}

__device__ __forceinline__ long long scan256(long long v, long long* sh, long long& total)
{
    return scan_wg<256>(v, sh, total);
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
// Where the cut falls among values that are spread out, as along the iteration once
// the volume has settled, the first digit holds some thousand points: they are listed
// and one workgroup ends the search among them.  Where it falls in the bulk (rough
// data whose domains diffuse away) the digit holds a large part of the field, which one
// workgroup would read again for every digit.  Above SEL_LIST_LDS points nothing is
// listed; the same launches take one more digit of SEL_BITS2 bits over the whole grid
// and, of as many points again, a third, and only the points of these digits are read
// by the one workgroup.  One iteration of 2048^2, n = 2 in float, 2 % of the points
// flipped at random: 0.60 ms, listing them all 19.6, by the general passes 0.63; with
// every value equal the selection alone takes 0.6 ms.
constexpr unsigned SEL_LIST_LDS = 8192;
constexpr int SEL_BITS2 = 13;
constexpr int SEL_NTF = 512;  // threads of sel_finish: large lists 6 to 10 % faster than with 256 or 1024, small ones alike
constexpr int SEL_NB2 = 1 << SEL_BITS2;
static_assert(SEL_NB2 + (1 << SEL_BITS) == SEL_HIST2, "the second and the third histogram");

// Search of a histogram of per * NT bins, from the top: the digit at which the running
// count reaches need, the rank within it and its points.  c: the thread's bins, the
// first at hi, downwards.  Every thread calls it.
template <int NT, int per>
__device__ __forceinline__ void sel_pick(const unsigned (&c)[per], int hi, long long need, long long* sh, int& s_digit,
                                            long long& s_need, unsigned& s_count)
{
    long long sum = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) sum += c[i];
    long long total;
    const long long incl = scan_wg<NT>(sum, sh, total);
    const long long excl = incl - sum;
    if (excl < need && need <= incl) {  // exactly one thread
        long long acc = excl;
        int d = hi;
        unsigned n = 0;
#pragma unroll
        for (int i = 0; i < per; ++i) {
            n = c[i];
            if (acc + (long long)c[i] >= need) {
                d = hi - i;
                break;
            }
            acc += c[i];
        }
        s_digit = d;
        s_need = need - acc;
        s_count = n;
    }
    __syncthreads();
}

// The values of a chunk (NT threads), every load in flight at once.
template <int NT, typename T>
__device__ __forceinline__ void sel_load(const T* v, int64_t x0, int64_t npts, T (&val)[SEL_CHUNK / NT])
{
#pragma unroll
    for (int k = 0; k < SEL_CHUNK / NT; ++k) {
        const int64_t x = x0 + (int64_t)k * NT;
        val[k] = x < npts ? v[x] : (T)0;
    }
}

// Appends the chunk's points with (key >> shift) == pre to the field's list, in no
// particular order.  Every thread calls it; s_cnt is zero before.
template <int NT, typename T>
__device__ __forceinline__ void sel_append(const SelListArgs& la, int b, const T (&val)[SEL_CHUNK / NT], int64_t x0,
                                           int shift, unsigned long long pre, unsigned& s_cnt, unsigned& s_base)
{
    const int64_t npts = la.s.npts;
    unsigned mine = 0;
#pragma unroll
    for (int k = 0; k < SEL_CHUNK / NT; ++k)
        mine += (x0 + (int64_t)k * NT < npts && (vp_key(val[k]) >> shift) == pre) ? 1u : 0u;
    unsigned at = mine ? atomicAdd(&s_cnt, mine) : 0u;
    __syncthreads();
    if (s_cnt == 0u) return;  // uniform
    if (threadIdx.x == 0) s_base = atomicAdd(la.count + b, s_cnt);
    __syncthreads();
    at += s_base;
    unsigned long long* lk = la.key + (size_t)b * npts;
    unsigned* li = la.idx + (size_t)b * npts;
#pragma unroll
    for (int k = 0; k < SEL_CHUNK / NT; ++k) {
        const int64_t x = x0 + (int64_t)k * NT;
        const unsigned long long key = vp_key(val[k]);
        if (x < npts && (key >> shift) == pre) {
            lk[at] = key;
            li[at] = (unsigned)x;
            ++at;
        }
    }
}

// The digit holding the cut, found by every workgroup for itself from the
// histogram (8 KB; one launch fewer than a pick kernel), then the chunk's points
// of that digit listed, or their next digit added to the second histogram.
template <typename T>
__global__ void __launch_bounds__(256) sel_list(const SelListArgs la, int shift)
{
    const SelArgs& a = la.s;
    __shared__ long long sh[4];
    __shared__ long long s_need;
    __shared__ int s_digit;
    __shared__ unsigned s_count, s_cnt, s_base;
    __shared__ unsigned h2[SEL_NB2];
    const int b = blockIdx.y, tid = threadIdx.x;
    const long long np = a.nplus[b];
    VpSel* st = a.st + b;
    if (blockIdx.x == 0 && tid == 0) la.clear[b] = 0u;
    if (np <= 0 || np >= a.npts) {  // uniform
        if (blockIdx.x == 0 && tid == 0) {
            st->mode = np <= 0 ? VS_NONE : VS_ALL;
            st->kstar = 0ull;
            st->need = 0;
            st->ties = 0;
            st->istar = -1;
            la.over[b] = 0u;
        }
        return;
    }
    // the chunk's loads in flight while the histogram is scanned
    const T* v = reinterpret_cast<const T*>(a.dE) + (size_t)b * a.npts;
    const int64_t x0 = (int64_t)blockIdx.x * SEL_CHUNK + tid;
    T val[SEL_PER];
    sel_load<256>(v, x0, a.npts, val);
    const unsigned* g = a.hist + (size_t)b * (1 << SEL_BITS);
    constexpr int per = (1 << SEL_BITS) / 256;
    const int hi = (1 << SEL_BITS) - 1 - tid * per;
    unsigned c[per];
#pragma unroll
    for (int i = 0; i < per; ++i) c[i] = g[hi - i];
    if (tid == 0) s_cnt = 0u;
    sel_pick<256>(c, hi, np, sh, s_digit, s_need, s_count);
    const unsigned long long digit = (unsigned long long)s_digit;
    const bool over = s_count > SEL_LIST_LDS;
    if (blockIdx.x == 0 && tid == 0) {
        st->kstar = digit << shift;
        st->need = s_need;
        st->mode = VS_SEARCH;
        st->istar = -1;
        la.over[b] = over ? 1u : 0u;
    }
    if (!over) {  // uniform
        sel_append<256>(la, b, val, x0, shift, digit, s_cnt, s_base);
        return;
    }
    for (int i = tid; i < SEL_NB2; i += 256) h2[i] = 0u;
    __syncthreads();
    unsigned bin = 0u, run = 0u;  // equal digits that follow each other count once, as in sel_hist
#pragma unroll
    for (int k = 0; k < SEL_PER; ++k) {
        const unsigned long long key = vp_key(val[k]);
        if (x0 + (int64_t)k * 256 < a.npts && (key >> shift) == digit) {
            const unsigned d = (unsigned)(key >> (shift - SEL_BITS2)) & (unsigned)(SEL_NB2 - 1);
            if (run && d != bin) {
                atomicAdd(&h2[bin], run);
                run = 0u;
            }
            bin = d;
            ++run;
        }
    }
    if (run) atomicAdd(&h2[bin], run);
    __syncthreads();
    unsigned* g2 = la.hist2 + (size_t)b * SEL_HIST2;
    for (int i = tid; i < SEL_NB2; i += 256)
        if (h2[i]) atomicAdd(&g2[i], h2[i]);
}

// The index of the rank-th point (in index order) with key ks, by one workgroup: counts
// per chunk, a wave each, then a walk through the chunk that holds it.
template <int NT, typename T>
__device__ __forceinline__ long long sel_tie_index(const SelArgs& a, const T* v, unsigned long long ks, long long rank,
                                                   unsigned* cnt, long long* sh)
{
    __shared__ long long s_chunk, s_rank, s_index;
    const int tid = threadIdx.x, lane = tid & 63;
    const int chunks = (int)a.chunks;
    for (int c = tid >> 6; c < chunks; c += NT / 64) {
        unsigned long long n = 0;
        constexpr int U = 32;  // loads in flight
        for (int k0 = 0; k0 < SEL_CHUNK / 64; k0 += U) {
            T val[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int64_t x = (int64_t)c * SEL_CHUNK + (k0 + k) * 64 + lane;
                val[k] = v[x < a.npts ? x : a.npts - 1];
            }
#pragma unroll
            for (int k = 0; k < U; ++k)
                n += ((int64_t)c * SEL_CHUNK + (k0 + k) * 64 + lane < a.npts && vp_key(val[k]) == ks) ? 1ull : 0ull;
        }
        n = wave_sum(n);
        if (lane == 0) cnt[c] = (unsigned)n;
    }
    if (tid == 0) {
        s_chunk = 0;
        s_rank = rank;
        s_index = -1;
    }
    __syncthreads();
    const int per = (chunks + NT - 1) / NT, c0 = tid * per;
    long long sum = 0, total;
    for (int c = c0; c < c0 + per && c < chunks; ++c) sum += cnt[c];
    long long incl = scan_wg<NT>(sum, sh, total);
    long long acc = incl - sum;
    if (acc < rank && rank <= incl)
        for (int c = c0; c < c0 + per && c < chunks; ++c) {
            if (acc + cnt[c] >= rank) {
                s_chunk = c;
                s_rank = rank - acc;
                break;
            }
            acc += cnt[c];
        }
    __syncthreads();
    constexpr int P = SEL_CHUNK / NT;  // neighbouring points of a thread
    const int64_t x0 = s_chunk * SEL_CHUNK + (int64_t)tid * P;
    const long long want = s_rank;
    bool eq[P];
    sum = 0;
#pragma unroll
    for (int k = 0; k < P; ++k) {
        eq[k] = x0 + k < a.npts && vp_key(x0 + k < a.npts ? v[x0 + k] : (T)0) == ks;
        sum += eq[k] ? 1 : 0;
    }
    incl = scan_wg<NT>(sum, sh, total);
    acc = incl - sum;
#pragma unroll
    for (int k = 0; k < P; ++k)
        if (eq[k] && ++acc == want) s_index = x0 + k;
    __syncthreads();
    return s_index;
}

// The end of the search among the listed points, by one workgroup per field:
// digits of SEL_BITS bits of the key below the ones found, then, when only some of
// the points with the last key are selected, of the index from the lower end.
// The list is copied to LDS.  Leaves the histograms and the count at zero.
// Where sel_list took the second histogram, every workgroup of the field finds its
// digit, lists the chunks' points of both digits and, where these are many too, adds
// their next bits to a third histogram; the workgroup that finishes last ends the
// search.  The others' list entries and counts are made visible to it by the
// device-scope fences on both sides of the finished-workgroup counter.  In float the
// three digits are the whole key.  In double a list of more than SEL_LIST_LDS points is
// read by that one workgroup, from where its keys first differ: points whose Delta E
// agree in 35 bits.
template <typename T>
__global__ void __launch_bounds__(SEL_NTF) sel_finish(const SelListArgs la, int shift0, int index_bits)
{
    constexpr int NT = SEL_NTF;
    const SelArgs& a = la.s;
    __shared__ long long sh[NT / 64];
    __shared__ unsigned h[1 << SEL_BITS];
    __shared__ unsigned long long lkey[SEL_LIST_LDS];
    __shared__ unsigned lidx[SEL_LIST_LDS];
    __shared__ unsigned long long s_pre, s_and, s_or;
    __shared__ long long s_need;
    __shared__ unsigned s_cnt, s_base, s_last;
    __shared__ int s_digit;
    const int b = blockIdx.y, tid = threadIdx.x;
    VpSel* st = a.st + b;
    const long long np = a.nplus[b];
    const bool none = np <= 0 || np >= a.npts;  // decided by sel_list, nothing listed
    const bool over = !none && la.over[b] != 0u;
    if (blockIdx.x > 0 && !over) return;  // uniform
    const T* v = reinterpret_cast<const T*>(a.dE) + (size_t)b * a.npts;
    unsigned* g = a.hist + (size_t)b * (1 << SEL_BITS);
    unsigned long long pre = st->kstar;
    int low = shift0;  // key bits below are still open
    unsigned M;
    if (!over) {
        M = la.count[b];
        for (int i = tid; i < (1 << SEL_BITS); i += NT) g[i] = 0u;
        if (none) return;
        __syncthreads();  // every wave has read the count, which is cleared below
        if (tid == 0) {
            s_need = st->need;
            s_cnt = M;
        }
    } else {
        unsigned *g2 = la.hist2 + (size_t)b * SEL_HIST2, *g3 = g2 + SEL_NB2;
        low -= SEL_BITS2;
        constexpr int per = SEL_NB2 / NT;
        const int hi = SEL_NB2 - 1 - tid * per;
        unsigned c[per];
#pragma unroll
        for (int i = 0; i < per; ++i) c[i] = g2[hi - i];
        sel_pick<NT>(c, hi, st->need, sh, s_digit, s_need, s_cnt);
        M = s_cnt;
        pre |= (unsigned long long)s_digit << low;
        const bool third = M > SEL_LIST_LDS;
        const bool list = !third || sizeof(T) == 8;
        constexpr int bits3 = sizeof(T) == 8 ? SEL_BITS : 32 - SEL_BITS - SEL_BITS2;
        for (int i = tid; i < (1 << bits3); i += NT) h[i] = 0u;
        unsigned bin = 0u, run = 0u;
        for (int64_t ch = blockIdx.x; ch < a.chunks; ch += gridDim.x) {
            const int64_t x0 = ch * SEL_CHUNK + tid;
            T val[SEL_CHUNK / NT];
            sel_load<NT>(v, x0, a.npts, val);
            __syncthreads();  // s_cnt and s_base have been read; h is clear
            if (tid == 0) s_last = 0u;
            __syncthreads();
            if (list) sel_append<NT>(la, b, val, x0, low, pre >> low, s_last, s_base);
            if (!third) continue;
#pragma unroll
            for (int k = 0; k < SEL_CHUNK / NT; ++k) {
                const unsigned long long key = vp_key(val[k]);
                if (x0 + (int64_t)k * NT < a.npts && (key >> low) == (pre >> low)) {
                    const unsigned d = (unsigned)(key >> (low - bits3)) & ((1u << bits3) - 1u);
                    if (run && d != bin) {
                        atomicAdd(&h[bin], run);
                        run = 0u;
                    }
                    bin = d;
                    ++run;
                }
            }
        }
        if (run) atomicAdd(&h[bin], run);
        __syncthreads();
        if (third)
            for (int i = tid; i < (1 << bits3); i += NT)
                if (h[i]) atomicAdd(&g3[i], h[i]);
        __threadfence();
        __syncthreads();
        if (tid == 0) s_last = atomicAdd(a.done + b, 1u) == gridDim.x - 1 ? 1u : 0u;
        __syncthreads();
        if (s_last == 0u) return;  // uniform
        __threadfence();
        if (third) {
            constexpr int per3 = (1 << SEL_BITS) / NT;
            const int hi3 = (1 << SEL_BITS) - 1 - tid * per3;
            unsigned c3[per3];
#pragma unroll
            for (int i = 0; i < per3; ++i) c3[i] = g3[hi3 - i];
            sel_pick<NT>(c3, hi3, s_need, sh, s_digit, s_need, s_cnt);
            low -= bits3;
            pre |= (unsigned long long)s_digit << low;
        }
        for (int i = tid; i < (1 << SEL_BITS); i += NT) g[i] = 0u;
        for (int i = tid; i < SEL_HIST2; i += NT) g2[i] = 0u;
        if (tid == 0) a.done[b] = 0u;
    }
    const unsigned long long* gk = la.key + (size_t)b * a.npts;
    const unsigned* gi = la.idx + (size_t)b * a.npts;
    const bool lds = M <= SEL_LIST_LDS;
    if (lds)
        for (unsigned i = tid; i < M; i += NT) {
            lkey[i] = gk[i];
            lidx[i] = gi[i];
        }
    auto key_at = [&](unsigned i) { return lds ? lkey[i] : gk[i]; };
    if (tid == 0) {
        s_pre = pre;
        la.count[b] = 0u;
    }
    __syncthreads();
    constexpr int U = 8;  // loads in flight
    // visits the listed keys (or, with the LDS list, the indices) for which `in` holds
    auto visit = [&](auto value, auto in, auto use) {
        for (unsigned i0 = tid; i0 < M; i0 += U * NT) {
            decltype(value(0u)) x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned i = i0 + (unsigned)(u * NT);
                x[u] = value(i < M ? i : i0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned i = i0 + (unsigned)(u * NT);
                if (i < M && in(i, x[u])) use(x[u]);
            }
        }
    };
    // one digit: histogram of (value >> sh) over the points for which `in`
    // holds, then the digit at which the running count, from the top (down) or
    // the bottom, reaches s_need; s_need becomes the rank within it.  Equal digits that
    // follow each other in a thread count once (equal values: one bin for them all)
    auto digit = [&](auto value, auto in, int shift, int bits, bool down) -> int {
        const int nb = 1 << bits;
        for (int i = tid; i < nb; i += NT) h[i] = 0u;
        __syncthreads();
        unsigned bin = 0u, run = 0u;
        visit(value, in, [&](auto x) {
            const unsigned d = (unsigned)(x >> shift) & (unsigned)(nb - 1);
            if (run && d != bin) {
                atomicAdd(&h[bin], run);
                run = 0u;
            }
            bin = d;
            ++run;
        });
        if (run) atomicAdd(&h[bin], run);
        __syncthreads();
        constexpr int per = (1 << SEL_BITS) / NT;
        unsigned c[per];
#pragma unroll
        for (int i = 0; i < per; ++i) {
            const int o = tid * per + i;
            c[i] = o < nb ? h[down ? nb - 1 - o : o] : 0u;
        }
        sel_pick<NT>(c, (1 << SEL_BITS) - 1 - tid * per, s_need, sh, s_digit, s_need, s_cnt);
        const int o = (1 << SEL_BITS) - 1 - s_digit;  // bins counted from the end searched from
        return down ? nb - 1 - o : o;
    };
    while (low > 0 && s_need != (long long)s_cnt) {
        if (!lds) {
            // the bits that every candidate shares are known
            if (tid == 0) {
                s_and = ~0ull;
                s_or = 0ull;
            }
            __syncthreads();
            unsigned long long all = ~0ull, any = 0ull;
            const unsigned long long p = s_pre >> low;
            visit(key_at, [&](unsigned, unsigned long long k) { return (k >> low) == p; },
                  [&](unsigned long long k) {
                      all &= k;
                      any |= k;
                  });
            atomicAnd(&s_and, all);
            atomicOr(&s_or, any);
            __syncthreads();
            const unsigned long long diff = s_and ^ s_or;
            low = diff ? 64 - __clzll((long long)diff) : 0;
            const unsigned long long same = (s_and >> low) << low;
            __syncthreads();
            if (tid == 0) s_pre = same;
            __syncthreads();
            if (low == 0) break;  // uniform
        }
        const int bits = low < SEL_BITS ? low : SEL_BITS;
        const int top = low;
        low -= bits;
        const unsigned long long p = top < 64 ? s_pre >> top : 0ull;
        const int d = digit(key_at, [&](unsigned, unsigned long long k) { return top >= 64 || (k >> top) == p; }, low,
                            bits, true);
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
    long long istar;
    if (lds) {
        unsigned ipre = 0u;
        int ilow = index_bits;
        while (ilow > 0) {
            const int bits = ilow < SEL_BITS ? ilow : SEL_BITS;
            const int top = ilow;
            ilow -= bits;
            const unsigned p = ipre >> top;
            const int d = digit([&](unsigned i) { return lidx[i]; },
                                [&](unsigned i, unsigned x) { return lkey[i] == ks && (x >> top) == p; }, ilow, bits,
                                false);
            ipre |= (unsigned)d << ilow;
        }
        istar = (long long)ipre;
    } else {
        istar = sel_tie_index<NT>(a, v, ks, s_need, lidx, sh);
    }
    if (tid == 0) {
        st->kstar = ks;
        st->mode = VS_TIES_PART;
        st->istar = istar;
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
    if (a.s.chunks <= 0 || batch <= 0 || a.s.npts > (1ll << 31) || a.s.chunks > (int64_t)SEL_LIST_LDS)
        return hipErrorInvalidValue;  // (2-D plans have at most 1024 chunks)
    const dim3 gc((unsigned)a.s.chunks, (unsigned)batch), bl(256);
    // the workgroups that sel_finish has beside the first end at once as a rule
    const dim3 gf((unsigned)std::min<int64_t>(a.s.chunks, std::max(8, 256 / batch)), (unsigned)batch);
    const int shift = (prec == 0 ? 64 : 32) - SEL_BITS;
    int ib = 0;
    while ((1ll << ib) < a.s.npts) ++ib;
    if (prec == 0) {
        hipLaunchKernelGGL((sel_hist<double>), gc, bl, 0, st, a.s, shift, SEL_BITS, 0);
        hipLaunchKernelGGL((sel_list<double>), gc, bl, 0, st, a, shift);
        hipLaunchKernelGGL((sel_finish<double>), gf, dim3(SEL_NTF), 0, st, a, shift, ib);
    } else {
        hipLaunchKernelGGL((sel_hist<float>), gc, bl, 0, st, a.s, shift, SEL_BITS, 0);
        hipLaunchKernelGGL((sel_list<float>), gc, bl, 0, st, a, shift);
        hipLaunchKernelGGL((sel_finish<float>), gf, dim3(SEL_NTF), 0, st, a, shift, ib);
    }
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

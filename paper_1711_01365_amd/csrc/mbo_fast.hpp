// Band-limited passes of Algorithm 1 on the 2-D flat torus for gfx950: the
// diffusion step of Section 5.1 (FFT, multiply by exp(-4 pi^2 tau |k|^2),
// inverse FFT) and the projection of Lemma 1.1, in two kernels per iteration.
//
// Kept modes.  The heat symbol is a product over the axes of
// exp(-4 pi^2 tau k^2); along an axis of length N the host keeps |k| <= c,
// with c the smallest half-width whose discarded symbol mass
// sum_{k outside the kept box} exp(-4 pi^2 tau |k|^2) is at most eta.  A value
// of the diffused field then moves by at most eta * max|A| when those modes
// are dropped (|A^(k)| <= N^d max|A| for every mode), far below the rounding of
// the transforms themselves (eta = 1e-12 for float plans, 1e-20 for double
// plans).  The row pass therefore stores, for every row, only the row spectrum
// at kx = 0..c and kx = N-c..N-1, in W slots per row (slot w holds kx = w for
// w <= c and kx = N - W + w for w >= W - c; the slots between hold zeros), and
// the column pass transforms only those W columns.  With c >= N/2 nothing is
// dropped and W = N.
//
//   row_fast   one workgroup owns 512 points (512/L whole rows) or, for rows of
//              1024 and 2048 points, one row: the line groups of its packed
//              planes load their kept modes straight into the FFT register
//              layout (lane t holds x[t + e L/8]), inverse-FFT (inside one wave
//              for L <= 512, in L/512 waves or with workgroup exchanges beyond) and
//              leave the lines in LDS; 512 threads or more, one to
//              four points each, project (Lemma 1.1) with the det-sign,
//              fallback, non-finite and change diagnostics; the line groups
//              forward-FFT and store the kept modes.  Float plans with n = 3
//              run the Newton polar iteration on every point that is certainly
//              well conditioned (1/|A^{-1}|_F > sigma_fb) and queue the others
//              for the first wave done with its own points, which projects
//              them by Jacobi (and in double when sigma_min < sigma_fb) at
//              raised priority.
//   heat_fast  a tile of TX stored columns of one packed plane: thread (t, cc)
//              loads rows t + e L/8 of column cc (TX-wide coalesced segments),
//              forward FFT along the column with workgroup exchanges, Lyapunov
//              partial sum_k symbol |Z|^2 (Section 4), symbol multiply, inverse
//              FFT, store in place.
#pragma once

#include <type_traits>

#include "mbo_kernels.hpp"
#include "mbo_volume.hpp"

namespace mbo {

// Stored slot of row mode kx, or -1 when the mode is not kept.
__device__ __forceinline__ int band_slot(int kx, int L, int c, int W)
{
    if (kx <= c) return kx;
    if (kx >= L - c) return W - (L - kx);
    return -1;
}

// ---------------------------------------------------------------------------
// Float n = 3 Newton polar iteration (Higham, 1986), split so that the
// workgroup can decide which points it runs before iterating: the steps of
// polar_newton3 with hardware reciprocals.
// ---------------------------------------------------------------------------
struct Newton3 {
    float X[9], C[9];
    float det, cf2;
};

// True when the float test of newton3_certain proves sigma_min > thr;
// otherwise the point goes to the Jacobi route.
__device__ __forceinline__ bool newton3_init(const float* a, Newton3& s, float thr)
{
#pragma unroll
    for (int k = 0; k < 9; ++k) s.X[k] = a[k];
    cofactor3(s.X, s.C);
    s.det = s.X[0] * s.C[0] + s.X[1] * s.C[1] + s.X[2] * s.C[2];
    s.cf2 = 0.f;
#pragma unroll
    for (int k = 0; k < 9; ++k) s.cf2 += s.C[k] * s.C[k];
    return newton3_certain(s.X, s.C, s.det, s.cf2, thr);
}

__device__ __forceinline__ void newton3_run(Newton3& s, float* q, int& dsign)
{
    dsign = s.det >= 0.f ? 1 : -1;
    bool scaled = true;
#pragma unroll 1
    for (int it = 0; it < 16; ++it) {
        if (it > 0) {
            cofactor3(s.X, s.C);
            s.det = s.X[0] * s.C[0] + s.X[1] * s.C[1] + s.X[2] * s.C[2];
            s.cf2 = 0.f;
#pragma unroll
            for (int k = 0; k < 9; ++k) s.cf2 += s.C[k] * s.C[k];
        }
        float xf2 = 0.f;
#pragma unroll
        for (int k = 0; k < 9; ++k) xf2 += s.X[k] * s.X[k];
        // the stopping test of polar_newton3 (newton3_near_done)
        bool last = false;
        if (it > 0) newton3_near_done(xf2, scaled, last);
        // hardware reciprocal (about 1 ulp): the iteration corrects its own
        // rounding, and a relative error of one ulp in the step's two scalar
        // factors stays below the float rounding of the result
        const float idet = num<float>::rcp(s.det);
        const float zeta = scaled ? num<float>::sqrt_(num<float>::sqrt_(s.cf2) * (idet < 0.f ? -idet : idet) *
                                                      num<float>::rsq(xf2))
                                  : 1.0f;
        const float cx = 0.5f * zeta, cc = 0.5f * idet * num<float>::rcp(zeta);
#pragma unroll
        for (int k = 0; k < 9; ++k) s.X[k] = cx * s.X[k] + cc * s.C[k];
        if (last) break;
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) q[k] = s.X[k];
}

// ---------------------------------------------------------------------------
// Row pass
// ---------------------------------------------------------------------------

// (x, y) times i^p
template <typename T>
__device__ __forceinline__ void turn(T& x, T& y, int p)
{
    if (p & 1) {
        const T v = x;
        x = -y;
        y = v;
    }
    if (p & 2) {
        x = -x;
        y = -y;
    }
}

// Adds ((ax, ay) + (-1)^q (bx, by)) i^p to (x, y): output q of dft2 or, in two
// steps, of dft4, with its operations.
template <typename T>
__device__ __forceinline__ void first_stage(T& x, T& y, T ax, T ay, T bx, T by, int q, int p)
{
    T vx = (q & 1) ? ax - bx : ax + bx, vy = (q & 1) ? ay - by : ay + by;
    turn(vx, vy, p);
    x += vx;
    y += vy;
}

// go(integral_constant<log2L>) for the row lengths of the band-limited passes, 8 to 2048.
template <typename Go>
static inline hipError_t with_row_length(int log2L, Go go)
{
    switch (log2L) {
    case 3: return go(std::integral_constant<int, 3>());
    case 4: return go(std::integral_constant<int, 4>());
    case 5: return go(std::integral_constant<int, 5>());
    case 6: return go(std::integral_constant<int, 6>());
    case 7: return go(std::integral_constant<int, 7>());
    case 8: return go(std::integral_constant<int, 8>());
    case 9: return go(std::integral_constant<int, 9>());
    case 10: return go(std::integral_constant<int, 10>());
    case 11: return go(std::integral_constant<int, 11>());
    }
    return hipErrorInvalidValue;
}

// Shape of a row-pass workgroup: 512 points (512/L rows) for L <= 512, one row
// of L points otherwise; NP projection threads (PPT points each); the line
// groups of Tn threads run in ROUNDS rounds of G transforms over NT threads.  A
// line of up to 512 points is one transform of L/8 threads inside a wave.  A longer
// one is, with PARTS, the R = L/512 parts of fft_wave, a wave each, after the
// radix-R first stage that each wave takes from the whole line: no exchange crosses
// a wave, one workgroup barrier per round and direction in place of two per stage,
// the same values; otherwise one transform of L/8 threads with workgroup barriers.
// Row pass, whole -> parts: 512 x 2048, n = 3 in float 49 -> 45 us; 1024 x 1024,
// n = 4 84 -> 74; 256 x 1024, n = 3 in double 26.6 -> 24.8.  The other instances gain
// less (n = 2 24 -> 22, n = 3 1024 x 1024 57 -> 51) and would round their transforms in
// another order, which changes the det sign of a tied point now and then.
template <typename T, int n, int LOG2L>
struct RowFastShape {
    static constexpr int L = 1 << LOG2L;
    static constexpr bool PARTS =
        LOG2L >= 10 && (n == 4 || (n >= 2 && sizeof(T) == 8) || (n == 3 && LOG2L == 11));
    static constexpr int R = PARTS ? L / 512 : 1;
    static constexpr int Tn = L / R / 8;
    static constexpr int NN = n * n;
    static constexpr int PL = (NN + 1) / 2;
    static constexpr int RPW = L >= 512 ? 1 : 512 / L;
    static constexpr int P = RPW * L;
    static constexpr int LINES = RPW * PL;
    static constexpr bool WAVE_LINE = LOG2L <= 9;
    static constexpr bool HELPER = sizeof(T) == 4 && n == 3;
    // float n = 4: points below sigma_fb are queued and re-projected in double
    // after the pass's loop (the double Jacobi inside the loop would spill)
    static constexpr bool DEFER4 = sizeof(T) == 4 && n == 4;
    // long rows: at most 768 threads for float n = 3 (twelve waves, a budget of
    // 168 registers for the queued points' double Jacobi), else 1024
    static constexpr int NTMAX = HELPER ? 768 : 1024;
    static constexpr int NT_LINES = LINES * R * Tn < NTMAX / (R * Tn) * (R * Tn) ? LINES * R * Tn
                                                                                  : NTMAX / (R * Tn) * (R * Tn);
    static constexpr int NT = WAVE_LINE ? 512 : (NT_LINES > 512 ? NT_LINES : 512);
    static constexpr int G = NT / Tn;  // transforms per round: whole lines (R divides G)
    static constexpr int ROUNDS = (LINES * R + G - 1) / G;
    static_assert(G % R == 0, "a round transforms whole lines");
    static constexpr int THREADS = NT;
    // projection threads: 512, or every thread of a long row's workgroup where
    // that leaves each fewer points (1024 points over 1024 threads at n = 4, 2048
    // over 768 at n = 3); where it does not (1024 over 640) the waves beyond the
    // 512 threads stay free for the queued points.  Four iterations of
    // 2048 x 2048 3 x 3 fields take 1129 us with 768 projecting threads, 1152 with
    // 512; ten of twelve fields of up to 1024 x 1024, n = 2..4, 4314 us and 4416.
    static constexpr int NP = (P + THREADS - 1) / THREADS < P / 512 ? THREADS : 512;
    static constexpr int PPT = (P + NP - 1) / NP;
    static constexpr int LP = L + L / 8;  // padded LDS line
    static constexpr size_t LDS_LINES = (size_t)LINES * LP * 2 * sizeof(T);
    // the twiddle table staged in LDS, where it fits beside the lines and the
    // static arrays (the queue, at most 4 KiB; 12 KiB are reserved): one load
    // per thread instead of 7 per radix-8 stage
    static constexpr size_t TW_BYTES = (size_t)L * 2 * sizeof(T);
    static constexpr bool TW_LDS = LDS_LINES + TW_BYTES + 12288 <= 163840;
    static constexpr size_t LDS = LDS_LINES + (TW_LDS ? TW_BYTES : 0);
    // waves per SIMD the instance is compiled for: two 512-point workgroups
    // (eight waves each, two per SIMD) per CU for short rows, one long-row
    // workgroup.  The register budget this leaves (128) holds the queued
    // points' double Jacobi without spilling: any scratch use would delay the
    // launch of the workgroups, and a ninth wave per workgroup would leave
    // room for only one of them per CU at that budget.  Double n = 4 does not
    // fit it (520 bytes of scratch): rows of 512 points run one workgroup per CU with 252 registers
    // instead (512^2, six steps: 482 us, with scratch 506; 1024 x 512 875 and 947);
    // shorter rows, whose workgroups end at more uneven times, keep two (1024 x
    // 256: 662 us, alone 688; 64^3, four steps: 525 and 548).
    static constexpr int WAVES = WAVE_LINE ? (sizeof(T) == 8 && n == 4 && LOG2L == 9 ? 2 : 4) : (THREADS + 255) / 256;
};

// What the points of a row pass go through between the two line transforms:
// FM_ITER the steps that the flags name (projection, load, store), FM_VJP the
// projection's vector-Jacobian product with the cotangent field a.Gin, FM_VKEY
// the projection with Delta E of the volume-preserving step into a.vde, FM_RELAX
// the reaction step of the relaxed flows (GD-1 by the projection of FM_ITER), FM_REDO
// nothing (the forward transform of the field's rows into a.Zout).
enum { FM_ITER = 0, FM_VJP = 1, FM_VKEY = 2, FM_RELAX = 3, FM_REDO = 4 };

template <typename T, int n, int LOG2L, bool PM, int MODE>
__device__ __forceinline__ void row_fast_body(const FastRowArgs& a, unsigned group)
{
    typedef RowFastShape<T, n, LOG2L> S;
    constexpr int NN = S::NN, PL = S::PL, L = S::L, Tn = S::Tn, RPW = S::RPW, LP = S::LP;
    constexpr int G = S::G, ROUNDS = S::ROUNDS, NT = S::NT, PPT = S::PPT, NP = S::NP;
    constexpr bool HELPER = S::HELPER;
    typedef typename cx<T>::type C;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* lr = reinterpret_cast<T*>(smem_raw);
    T* li = lr + (size_t)S::LINES * LP;
    __shared__ unsigned short fq[(HELPER || S::DEFER4 || ((MODE == FM_VJP || MODE == FM_VKEY) && n == 3)) ? S::P : 1];
    __shared__ int fq_n, fq_claim;
    // rows of at most 512 points (every wave holds points): the last wave's
    // Newton points, handed to the other waves when it runs the queue
    constexpr bool SPLIT = HELPER && S::THREADS == 512 && S::PPT == 1;
    __shared__ int hq[SPLIT ? 64 : 1];
    __shared__ int hq_n, hq_claim;
    __shared__ unsigned long long wg_cnt[2];

    const int flags = MODE == FM_REDO ? RF_LOAD_REAL | RF_FORWARD : a.flags;
    const int b = blockIdx.y;
    const int tid = threadIdx.x;
    if (tid == 0) {
        fq_n = 0;
        fq_claim = 0;
        hq_n = 0;
        hq_claim = 0;
        wg_cnt[0] = 0;
        wg_cnt[1] = 0;
    }
    const int64_t npts = a.npts;
    const int W = a.W, c = a.band;
    // PM: spectra stored plane by plane (a.plane_major, the 3-D layout).
    constexpr bool pm = PM;
    // Plane by plane, a workgroup's loads and stores of one mode cover RPW
    // consecutive rows, part of a cache line: the eight XCDs (own L2 each) then
    // take contiguous runs of row groups, so that the groups sharing a line
    // run on one XCD.
    const int64_t nwgx = gridDim.x;
    const int64_t row0 = RPW * (((nwgx & 7) || !pm) ? (int64_t)group
                                                    : (int64_t)(blockIdx.x & 7) * (nwgx >> 3) + (blockIdx.x >> 3));
    C* Zb = reinterpret_cast<C*>(a.Z) + (size_t)b * PL * a.rows * W;
    C* Zo = MODE == FM_VKEY || MODE == FM_REDO ? reinterpret_cast<C*>(a.Zout) + (size_t)b * PL * a.rows * W : Zb;

    // Every global load that does not depend on another is issued first (the
    // kept modes of the first round of lines, the twiddles, the previous det
    // signs, the stop mark): at the start of a launch each round trip to memory
    // is a cold miss, and none of them waits for another.
    const int g = tid / Tn, t = tid - (tid / Tn) * Tn;
    const int pt = lds_pad(t);
    const bool fft_thread = tid < NT;
    constexpr int R = S::R, LOG2S = S::PARTS ? 9 : LOG2L;  // log2 of a transform's points
    constexpr bool IMF = n < 4;  // the order in which the whole-line transform of the instance is compiled
    const int q = g & (R - 1);                                 // its part of the line (R divides G)
    Twiddles<T, LOG2L> tw;
    T r[1][8], im[1][8];
    // Transform j is part q of line j / R; line j is row rl, packed plane
    // pl of the workgroup (LDS line rl*PL + pl).  Spectra are stored row by row
    // (Z[plane][row][w]) or, for the 3-D plane pass, plane by plane
    // (Z[plane][w][row]): there the lines of one plane go to neighbouring groups, so
    // that a wave's stores of one mode cover consecutive rows.
    auto line_of = [&](int j, int& rl, int& pl) {
        if (pm) {
            rl = j % RPW;
            pl = j / RPW;
        } else {
            rl = j / PL;
            pl = j - (j / PL) * PL;
        }
    };
    auto zat = [&](int pl, int64_t row, int w) -> size_t {
        return pm ? ((size_t)pl * W + w) * a.rows + row : ((size_t)pl * a.rows + row) * W + w;
    };
    auto load_line = [&](int j) {
        int rl, pl;
        line_of(j / R, rl, pl);
        const bool live = j < S::LINES * R && row0 + rl < a.rows;
        const int64_t row = live ? row0 + rl : 0;
        if (!S::PARTS || c < 256) {
            // the one kept mode of those at distance 512
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int kx = t + e * Tn;
                const int w = band_slot(!S::PARTS || kx <= c ? kx : kx + 512 * (R - 1), L, c, W);
                C v;
                if (live && w >= 0) v = Zb[zat(pl, row, w)];
                else { v.x = 0; v.y = 0; }
                r[0][e] = v.x;
                im[0][e] = v.y;
            }
        } else if (R == 4 && n < 4 && c < 512) {
            // the modes of the lowest and of the highest quarter
            C hv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int kx = t + e * Tn, kh = kx + 512 * (R - 1);
                const int w = kx <= c ? kx : -1, wh = kh >= L - c ? W - (L - kh) : -1;
                C v;
                if (live && w >= 0) v = Zb[zat(pl, row, w)];
                else { v.x = 0; v.y = 0; }
                if (live && wh >= 0) hv[e] = Zb[zat(pl, row, wh)];
                else { hv[e].x = 0; hv[e].y = 0; }
                r[0][e] = v.x;
                im[0][e] = v.y;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                turn(hv[e].x, hv[e].y, 3 * q);
                r[0][e] += hv[e].x;
                im[0][e] += hv[e].y;
            }
        } else {
            // every other case: the first stage (output q of dft2 or dft4) at the loads
            C hv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) r[0][e] = im[0][e] = 0;
#pragma unroll 1
            for (int m = 0; m < R / 2; ++m) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int kx = t + e * Tn + 512 * m;
                    const int w = band_slot(kx, L, c, W), wh = band_slot(kx + 512 * (R / 2), L, c, W);
                    C v;
                    if (live && w >= 0) v = Zb[zat(pl, row, w)];
                    else { v.x = 0; v.y = 0; }
                    if (live && wh >= 0) hv[e] = Zb[zat(pl, row, wh)];
                    else { hv[e].x = 0; hv[e].y = 0; }
                    first_stage(r[0][e], im[0][e], v.x, v.y, hv[e].x, hv[e].y, q, q * m);
                }
            }
        }
    };
    if ((flags & RF_INVERSE) && fft_thread) load_line(g);
    const C* twg = reinterpret_cast<const C*>(a.tw);
    C* twl = reinterpret_cast<C*>(smem_raw + S::LDS_LINES);
    if constexpr (S::TW_LDS) {
        if (flags & (RF_INVERSE | RF_FORWARD)) {
            for (int m = tid; m < L; m += S::THREADS) twl[m] = twg[m];
            __syncthreads();
        }
    }
    if (fft_thread && (flags & RF_INVERSE)) load_twiddles<T, LOG2L>(tw, S::TW_LDS ? twl : twg, R * t + q);
    int8_t* sgn = a.sgn + (size_t)b * npts;
    // previous det signs of the thread's points, a byte each (a register, not
    // an array: the projection loops index it at run time)
    unsigned s_old = 0;
#pragma unroll
    for (int pp = 0; pp < PPT; ++pp) {
        const int idx = pp * NP + tid;
        const bool live = tid < NP && idx < S::P && row0 + (idx >> LOG2L) < a.rows;
        const int8_t so = (live && (flags & RF_SIGN)) ? sgn[(row0 + (idx >> LOG2L)) * L + (idx & (L - 1))] : (int8_t)0;
        s_old |= (unsigned)(uint8_t)so << (8 * pp);
    }
    const int stop = (flags & RF_CHECK_STOP) ? a.stop_iter[b] : a.iter;

    // ---- phase 1: inverse FFT of each line, natural order into LDS
    if (flags & RF_INVERSE) {
#pragma unroll 1
        for (int rd = 0; rd < ROUNDS; ++rd) {
            const int j = rd * G + g;
            const bool act = fft_thread && j < S::LINES * R;
            if (rd > 0 && fft_thread) load_line(j);
            int rl, pl;
            line_of(j / R, rl, pl);
            const int lj = act ? rl * PL + pl : 0;
            T* lrj = lr + (size_t)lj * LP;
            T* lij = li + (size_t)lj * LP;
            const int part = q * (LP / R);  // the exchanges of part q
            if constexpr (S::WAVE_LINE || S::PARTS) {
                if (act) {
                    if (S::PARTS && c < 256) {
                        // output q of the first stage, of one nonzero input
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (t + e * Tn > c) turn(r[0][e], im[0][e], (4 / R) * q * (R - 1));
                    }
                    // with c < Tn only the loads e = 0, 7 hold kept modes (float, n <= 3:
                    // the double and n = 4 instances have no registers to spare for a
                    // second copy of the transform)
                    if constexpr (sizeof(T) == 4 && n <= 3 && FftShape<LOG2S>::R0 == 1 && FftShape<LOG2S>::NST > 1) {
                        if (c < Tn) fft_wave<T, +1, LOG2S, 0, FFT_IN07, LOG2L>(r[0], im[0], lrj + part, lij + part, t, tw, true);
                        else fft_wave<T, +1, LOG2S, 0, FFT_FULL, LOG2L>(r[0], im[0], lrj + part, lij + part, t, tw, true);
                    } else {
                        fft_wave<T, +1, LOG2S, 0, FFT_FULL, LOG2L>(r[0], im[0], lrj + part, lij + part, t, tw, true);
                    }
                    wave_lds_sync();  // the transform's last exchange has been read
                }
                if constexpr (S::PARTS) __syncthreads();  // by every wave of the line
            } else {
                fft_lines<T, +1, 1, LOG2L>(r, im, lrj, lij, 0, 1, 0, t, tw, act);
                __syncthreads();  // the line's last exchange has been read
            }
            if (act) {
                const int o = R * t + q, po = lds_pad(o);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    lrj[lds_pad_at<R * Tn>(o, po, e)] = r[0][e];
                    lij[lds_pad_at<R * Tn>(o, po, e)] = im[0][e];
                }
            }
        }
    }
    // a field that already stopped is left alone (uniform per workgroup; the
    // loads above only read)
    if (stop < a.iter) return;

    // ---- phase 2: PPT points per projection thread
    // the field's pointer from its device word where there is one (a captured
    // iteration then serves any field buffer)
    T* Aout = reinterpret_cast<T*>(a.slot ? *a.slot : a.Aout) + field_base(a.foff, b, NN * npts);
    unsigned long long nflip = 0, nfb = 0, nbad = 0;
    double dmax = 0.0;
    const bool fallback = (flags & RF_FALLBACK) != 0;
    auto point_of = [&](int idx, int64_t& xp, T*& lrq, T*& liq) {
        const int rq = idx >> LOG2L, xq = idx & (L - 1);
        xp = (row0 + rq) * L + xq;
        lrq = lr + (size_t)rq * PL * LP + lds_pad(xq);
        liq = li + (size_t)rq * PL * LP + lds_pad(xq);
        return idx < S::P && row0 + rq < a.rows;
    };

    // diagnostics and write-back of a projected point (LDS slot at lrq/liq)
    auto finish = [&](int64_t xp, T* lrq, T* liq, T (&qv)[NN], int ds, int8_t so) {
        if constexpr (MODE == FM_RELAX) {
            // GD-1: N(A) = U (Sigma - I) V^t = A - U V^t, the point is still in LDS
            const T rc = (T)a.relax_c;
#pragma unroll
            for (int k = 0; k < NN; ++k) {
                const T av = (k & 1) ? liq[(k >> 1) * LP] : lrq[(k >> 1) * LP];
                qv[k] = av - rc * (av - qv[k]);
            }
        }
        if (flags & RF_SIGN) {
            nflip += (so != (int8_t)ds) ? 1ull : 0ull;
            sgn[xp] = (int8_t)ds;
        }
        if (flags & RF_TRACK) {
#pragma unroll
            for (int k = 0; k < NN; ++k) {
                const double dv = fabs((double)qv[k] - (double)Aout[(int64_t)k * npts + xp]);
                dmax = dv > dmax ? dv : dmax;
            }
        }
        if (flags & RF_STORE_REAL) {
#pragma unroll
            for (int k = 0; k < NN; ++k) Aout[(int64_t)k * npts + xp] = qv[k];
        }
#pragma unroll
        for (int k = 0; k < NN; ++k) {
            if (k & 1) liq[(k >> 1) * LP] = qv[k];
            else lrq[(k >> 1) * LP] = qv[k];
        }
        if (NN & 1) liq[(NN >> 1) * LP] = (T)0;
    };
    auto load_point = [&](const T* lrq, const T* liq, T (&av)[NN]) {
#pragma unroll
        for (int k = 0; k < NN; ++k) av[k] = (k & 1) ? liq[(k >> 1) * LP] : lrq[(k >> 1) * LP];
    };

    if (flags & RF_LOAD_REAL) {
        // forward transform of a real field: the points' entries from A
        const T* A = (a.slot ? Aout : reinterpret_cast<const T*>(a.Ain) + field_base(a.foff, b, NN * npts));
#pragma unroll 1
        for (int pp = 0; pp < PPT; ++pp) {
            int64_t xp;
            T *lrq, *liq;
            if (tid < NP && point_of(pp * NP + tid, xp, lrq, liq)) {
                T av[NN];
#pragma unroll
                for (int k = 0; k < NN; ++k) av[k] = A[(int64_t)k * npts + xp];
                if (flags & RF_SIGN_INIT) sgn[xp] = det_n<T, n>(av) >= (T)0 ? 1 : -1;
#pragma unroll
                for (int k = 0; k < NN; ++k) {
                    if (k & 1) liq[(k >> 1) * LP] = av[k];
                    else lrq[(k >> 1) * LP] = av[k];
                }
                if (NN & 1) liq[(NN >> 1) * LP] = (T)0;
            }
        }
    }
    __syncthreads();

    if constexpr (MODE == FM_VJP) {
        // Points certainly well conditioned (n = 3) or in closed form (n = 2):
        // polar_vjp_newton3 / polar_vjp2_fb; the others (n = 3) are queued for the
        // first wave done, which runs Jacobi (in double below sigma_fb).
        const T* G = reinterpret_cast<const T*>(a.Gin) + field_base(a.foff, b, NN * npts);
        auto put = [&](T* lrq, T* liq, const T (&ov)[NN]) {
#pragma unroll
            for (int k = 0; k < NN; ++k) {
                if (k & 1) liq[(k >> 1) * LP] = ov[k];
                else lrq[(k >> 1) * LP] = ov[k];
            }
            if (NN & 1) liq[(NN >> 1) * LP] = (T)0;
        };
#pragma unroll 1
        for (int pp = 0; pp < PPT; ++pp) {
            int64_t xp;
            T *lrq, *liq;
            if (tid < NP && point_of(pp * NP + tid, xp, lrq, liq)) {
                T av[NN], gv[NN], ov[NN];
#pragma unroll
                for (int k = 0; k < NN; ++k) gv[k] = G[(int64_t)k * npts + xp];
                load_point(lrq, liq, av);
                if constexpr (n == 2) {
                    polar_vjp2_fb<T>(av, gv, ov, fallback, a.sigma_fb);
                    put(lrq, liq, ov);
                } else {
                    if (polar_vjp_newton3<T, 3>(av, gv, ov, a.sigma_fb)) {
                        put(lrq, liq, ov);
                    } else {
                        fq[atomicAdd(&fq_n, 1)] = (unsigned short)(pp * NP + tid);
                    }
                }
            }
        }
        if constexpr (n == 3) {
            __syncthreads();
            if (fq_n > 0) {  // uniform
                if (tid < 64) {
                    __builtin_amdgcn_s_setprio(3);
#pragma unroll 1
                    for (int qi = tid; qi < fq_n; qi += 64) {
                        int64_t xp;
                        T *lrq, *liq;
                        (void)point_of(fq[qi], xp, lrq, liq);
                        T av[NN], ov[NN];
                        load_point(lrq, liq, av);
                        polar_vjp3_fb<T>(av, G + xp, npts, ov, fallback, a.sigma_fb);
                        put(lrq, liq, ov);
                    }
                    __builtin_amdgcn_s_setprio(0);
                }
            }
        }
        __syncthreads();
    } else if constexpr (MODE == FM_VKEY) {
        // Q = U V^t of every point, Delta E = +-2 sigma_min with the sign bit
        // of det Q (also where sigma_min is 0: volume_fix reads the side there) and the
        // n values from which volume_fix forms the other candidate (vp_change).
        // Float points below sigma_fb are queued and done in double afterwards.
        T* vde = reinterpret_cast<T*>(a.vde) + (size_t)b * npts;
        T* vdir = reinterpret_cast<T*>(a.vdir) + (size_t)b * n * npts;
        auto key_out = [&](int64_t xp, T* lrq, T* liq, T (&qv)[NN], int ds, T smin) {
            vde[xp] = ds > 0 ? smin + smin : -(smin + smin);
            finish(xp, lrq, liq, qv, ds, (int8_t)0);
        };
        constexpr bool QUEUE = sizeof(T) == 4 && n >= 3;
#pragma unroll 1
        for (int pp = 0; pp < PPT; ++pp) {
            int64_t xp;
            T *lrq, *liq;
            if (tid < NP && point_of(pp * NP + tid, xp, lrq, liq)) {
                T av[NN], qv[NN];
                load_point(lrq, liq, av);
                nbad += all_finite<T, NN>(av) ? 0ull : 1ull;
                if constexpr (n <= 2) {
                    T tm[NN], de;
                    nfb += vp_point<T, n>(av, qv, tm, de, fallback, a.sigma_fb) ? 1ull : 0ull;
                    const bool plus = de >= (T)0;
                    if constexpr (n == 2) {
                        vdir[xp] = plus ? tm[0] : qv[0];
                        vdir[npts + xp] = plus ? tm[2] : qv[2];
                    }
                    if (!plus) {
#pragma unroll
                        for (int k = 0; k < NN; ++k) qv[k] = tm[k];
                    }
                    const T half = (de < (T)0 ? -de : de) * (T)0.5;
                    key_out(xp, lrq, liq, qv, plus ? 1 : -1, half);
                } else {
                    int ds;
                    T smin;
                    polar_jacobi<T, n>(av, qv, ds, smin, [&](const T(&W)[n][n], const T(&V)[n][n]) {
                        T v[n];
                        min_direction<T, n>(W, V, v);
#pragma unroll
                        for (int k = 0; k < n; ++k) vdir[k * npts + xp] = v[k];
                    });
                    if (QUEUE && fallback && (double)smin < a.sigma_fb)
                        fq[atomicAdd(&fq_n, 1)] = (unsigned short)(pp * NP + tid);
                    else
                        key_out(xp, lrq, liq, qv, ds, smin);
                }
            }
        }
        if constexpr (QUEUE) {
            __syncthreads();
            if (fq_n > 0 && tid < 64) {
                __builtin_amdgcn_s_setprio(3);
#pragma unroll 1
                for (int qi = tid; qi < fq_n; qi += 64) {
                    int64_t xp;
                    T *lrq, *liq;
                    (void)point_of(fq[qi], xp, lrq, liq);
                    float aq[NN], qv[NN];
                    load_point(lrq, liq, aq);
                    float V[n][n];
                    int ds;
                    float sm;
                    {
                        // float Jacobi again for its V (sigma_fb = inf: it stops there)
                        (void)polar_jacobi_f32_fb<n>(aq, qv, ds, V, INFINITY);
                        sm = (float)polar_jacobi_warm<n>(
                            aq, V, qv, ds, [&](const double(&Wd)[n][n], const double(&Vd)[n][n]) {
                                double v[n];
                                min_direction<double, n>(Wd, Vd, v);
#pragma unroll
                                for (int k = 0; k < n; ++k) vdir[k * npts + xp] = (T)v[k];
                            });
                    }
                    ++nfb;
                    key_out(xp, lrq, liq, qv, ds, sm);
                }
                __builtin_amdgcn_s_setprio(0);
            }
        }
        __syncthreads();
    } else if (MODE == FM_RELAX && a.relax_kind == 3) {
        // GD-3: N(A) = A (A^t A - I)
#pragma unroll 1
        for (int pp = 0; pp < PPT; ++pp) {
            int64_t xp;
            T *lrq, *liq;
            if (tid < NP && point_of(pp * NP + tid, xp, lrq, liq)) {
                T av[NN], m[NN];
                load_point(lrq, liq, av);
                nbad += all_finite<T, NN>(av) ? 0ull : 1ull;
#pragma unroll
                for (int i = 0; i < n; ++i)
#pragma unroll
                    for (int j = 0; j < n; ++j) {
                        T v = 0;
#pragma unroll
                        for (int k = 0; k < n; ++k) v += av[k * n + i] * av[k * n + j];
                        m[i * n + j] = v - (i == j ? (T)1 : (T)0);
                    }
                const T rc = (T)a.relax_c;
#pragma unroll
                for (int i = 0; i < n; ++i)
#pragma unroll
                    for (int j = 0; j < n; ++j) {
                        T v = 0;
#pragma unroll
                        for (int k = 0; k < n; ++k) v += av[i * n + k] * m[k * n + j];
                        v = av[i * n + j] - rc * v;
                        const int e = i * n + j;
                        if (e & 1) liq[(e >> 1) * LP] = v;
                        else lrq[(e >> 1) * LP] = v;
                        if (flags & RF_STORE_REAL) Aout[(int64_t)e * npts + xp] = v;
                    }
            }
        }
        __syncthreads();
    } else if (MODE == FM_RELAX || (flags & RF_PROJECT)) {
        if constexpr (HELPER) {
            // which points are certainly well conditioned: the Newton
            // iteration; the others are queued
            Newton3 ns;       // kept from the test when each thread has one point
            unsigned ok = 0;  // bit pp: point pp runs Newton
#pragma unroll 1
            for (int pp = 0; pp < PPT; ++pp) {
                int64_t xp;
                T *lrq, *liq;
                if (tid < NP && point_of(pp * NP + tid, xp, lrq, liq)) {
                    T av[NN];
                    load_point(lrq, liq, av);
                    nbad += all_finite<T, NN>(av) ? 0ull : 1ull;
                    if (newton3_init(av, ns, (float)a.sigma_fb)) {
                        ok |= 1u << pp;
                        // the last wave's Newton points, with their previous
                        // det sign, for the other waves to take over when it
                        // becomes the queue's wave
                        if (SPLIT && tid >= 512 - 64)
                            hq[atomicAdd(&hq_n, 1)] = (pp * NP + tid) | ((int)(uint8_t)(s_old >> (8 * pp)) << 16);
                    } else {
                        fq[atomicAdd(&fq_n, 1)] = (unsigned short)(pp * NP + tid);
                    }
                }
            }
            __syncthreads();
            // Queued points: Jacobi in float, and in double (warm-started from
            // the float right singular vectors) when sigma_min < sigma_fb, at
            // raised priority, one point per lane of the wave that runs them.
            auto run_queue = [&]() {
                __builtin_amdgcn_s_setprio(3);
                const int nq = fq_n;
                const int lane = tid & 63;
#pragma unroll 1
                for (int qi = lane; qi < nq; qi += 64) {
                    int64_t xp;
                    T *lrq, *liq;
                    (void)point_of(fq[qi], xp, lrq, liq);
                    float aq[NN], qv[NN];
                    load_point(lrq, liq, aq);
                    int ds;
                    if (fallback) {
                        float V[n][n];
                        if (polar_jacobi_f32_fb<n>(aq, qv, ds, V, a.sigma_fb)) {
                            polar_jacobi_warm<n>(aq, V, qv, ds);
                            ++nfb;
                        }
                    } else {
                        float smin;
                        polar_jacobi<float, n>(aq, qv, ds, smin);
                    }
                    finish(xp, lrq, liq, qv, ds, (flags & RF_SIGN) ? sgn[xp] : (int8_t)0);
                }
                __builtin_amdgcn_s_setprio(0);
            };
            // With every wave holding points (rows of at most 512 points) and a
            // non-empty queue, the last wave starts on the queue at once and
            // the first wave done with its own points takes the last wave's
            // Newton points: the queue's serial Jacobi chain then overlaps the
            // other waves' Newton iterations instead of following them.
            const bool split = SPLIT && fq_n > 0;
            const bool qwave = split && tid >= 512 - 64;
            if (tid < NP && !qwave) {
#pragma unroll 1
                for (int pp = 0; pp < PPT; ++pp) {
                    if (!(ok >> pp & 1u)) continue;
                    int64_t xp;
                    T *lrq, *liq;
                    (void)point_of(pp * NP + tid, xp, lrq, liq);
                    if constexpr (PPT > 1) {
                        T av[NN];
                        load_point(lrq, liq, av);
                        (void)newton3_init(av, ns, (float)a.sigma_fb);
                    }
                    T qv[NN];
                    int ds;
                    newton3_run(ns, qv, ds);
                    finish(xp, lrq, liq, qv, ds, (int8_t)(s_old >> (8 * pp)));
                }
            }
            if (split) {
                if (qwave) {
                    run_queue();
                } else {
                    // the last wave's Newton points, one per lane of the first
                    // wave(s) to get here (hq_n is final since the barrier)
#pragma unroll 1
                    for (;;) {
                        const int i = atomicAdd(&hq_claim, 1);
                        if (i >= hq_n) break;
                        const int e = hq[i];
                        int64_t xp;
                        T *lrq, *liq;
                        (void)point_of(e & 0xffff, xp, lrq, liq);
                        T av[NN];
                        load_point(lrq, liq, av);
                        Newton3 hs;
                        (void)newton3_init(av, hs, (float)a.sigma_fb);
                        T qv[NN];
                        int ds;
                        newton3_run(hs, qv, ds);
                        finish(xp, lrq, liq, qv, ds, (int8_t)(e >> 16));
                    }
                }
            } else {
                // The queued points go to the first wave done with its own
                // points (threads beyond the projection threads have none).  A wave of its own would cost the registers
                // that let two workgroups share a CU.
                int claim = 0;
                if ((tid & 63) == 0) claim = atomicAdd(&fq_claim, 1);
                claim = __shfl(claim, 0, 64);
                if (claim == 0) run_queue();
            }
        } else {
#pragma unroll 1
            for (int pp = 0; pp < PPT; ++pp) {
                int64_t xp;
                T *lrq, *liq;
                if (tid < NP && point_of(pp * NP + tid, xp, lrq, liq)) {
                    T av[NN], qv[NN];
                    load_point(lrq, liq, av);
                    nbad += all_finite<T, NN>(av) ? 0ull : 1ull;
                    int ds;
                    if constexpr (S::DEFER4) {
                        if (polar_newton<float, n>(av, qv, ds, (float)a.sigma_fb)) {
                            // well conditioned: Newton, no fallback
                        } else if (fallback) {
                            float V[n][n];
                            if (polar_jacobi_f32_fb<n>(av, qv, ds, V, a.sigma_fb)) {
                                fq[atomicAdd(&fq_n, 1)] = (unsigned short)(pp * NP + tid);
                                continue;
                            }
                        } else {
                            T smin;
                            project_point<T, n>(av, qv, ds, smin);
                        }
                    } else {
                        if (project_point_fb<T, n>(av, qv, ds, fallback, a.sigma_fb)) ++nfb;
                    }
                    finish(xp, lrq, liq, qv, ds, (int8_t)(s_old >> (8 * pp)));
                }
            }
            if constexpr (S::DEFER4) {
                // the queued points: float Jacobi again for its V, then the
                // double Jacobi warm-started from it
                if (fallback) {
                    __syncthreads();
                    const int nq = fq_n;
#pragma unroll 1
                    for (int qi = tid; qi < nq; qi += S::THREADS) {
                        int64_t xp;
                        T *lrq, *liq;
                        (void)point_of(fq[qi], xp, lrq, liq);
                        float aq[NN], qv[NN];
                        load_point(lrq, liq, aq);
                        float V[n][n];
                        int ds;
                        (void)polar_jacobi_f32_fb<n>(aq, qv, ds, V, a.sigma_fb);
                        polar_jacobi_warm<n>(aq, V, qv, ds);
                        ++nfb;
                        finish(xp, lrq, liq, qv, ds, (flags & RF_SIGN) ? sgn[xp] : (int8_t)0);
                    }
                }
            }
        }
        __syncthreads();
    } else if ((flags & (RF_INVERSE | RF_STORE_REAL)) == (RF_INVERSE | RF_STORE_REAL)) {
        // the transformed values as they are (a diffusion step without projection)
#pragma unroll 1
        for (int pp = 0; pp < PPT; ++pp) {
            int64_t xp;
            T *lrq, *liq;
            if (tid < NP && point_of(pp * NP + tid, xp, lrq, liq)) {
#pragma unroll
                for (int k = 0; k < NN; ++k)
                    Aout[(int64_t)k * npts + xp] = (k & 1) ? liq[(k >> 1) * LP] : lrq[(k >> 1) * LP];
            }
        }
    }

    // ---- phase 3: forward FFT of the lines, store the kept modes
    if (flags & RF_FORWARD) {
        // the twiddles again (from LDS or cache), into a fresh variable: the
        // values of phase 1 kept alive across the projection would raise its
        // register peak above what the kernel's occupancy allows
        Twiddles<T, LOG2L> tw3;
        if (fft_thread) load_twiddles<T, LOG2L>(tw3, S::TW_LDS ? twl : twg, R * t + q);
#pragma unroll 1
        for (int rd = 0; rd < ROUNDS; ++rd) {
            const int j = rd * G + g;
            const bool act = fft_thread && j < S::LINES * R;
            int rl, pl;
            line_of(j / R, rl, pl);
            const int lj = act ? rl * PL + pl : 0;
            T* lrj = lr + (size_t)lj * LP;
            T* lij = li + (size_t)lj * LP;
            const int part = q * (LP / R);
            T r3[1][8], im3[1][8];  // fresh, as tw3
            if (act) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int o = lds_pad_at<Tn>(t, pt, e);
                    r3[0][e] = lrj[o];
                    im3[0][e] = lij[o];
                    if constexpr (R > 1) {
                        constexpr int H = LP / 2;
                        T xr = r3[0][e], xi = im3[0][e];
                        r3[0][e] = im3[0][e] = 0;
                        first_stage(r3[0][e], im3[0][e], xr, xi, lrj[o + H], lij[o + H], q, 0);
                        if constexpr (R == 4)
                            first_stage(r3[0][e], im3[0][e], lrj[o + H / 2], lij[o + H / 2], lrj[o + 3 * H / 2],
                                        lij[o + 3 * H / 2], q, -q);
                    }
                }
            }
            if constexpr (S::WAVE_LINE || S::PARTS) {
                // every lane (of a line in parts, every wave) has read its elements
                // before the exchanges
                if constexpr (S::PARTS) __syncthreads();
                if (act) {
                    if constexpr (S::WAVE_LINE) wave_lds_sync();
                    // with c < R Tn only the modes e = 0, 7 are stored
                    if constexpr (sizeof(T) == 4 && n <= 3 && FftShape<LOG2S>::NST > 1) {
                        if (c < R * Tn) fft_wave<T, -1, LOG2S, 0, FFT_OUT07, LOG2L, IMF>(r3[0], im3[0], lrj + part, lij + part, t, tw3, true);
                        else fft_wave<T, -1, LOG2S, 0, FFT_FULL, LOG2L, IMF>(r3[0], im3[0], lrj + part, lij + part, t, tw3, true);
                    } else {
                        fft_wave<T, -1, LOG2S, 0, FFT_FULL, LOG2L, IMF>(r3[0], im3[0], lrj + part, lij + part, t, tw3, true);
                    }
                }
            } else {
                fft_lines<T, -1, 1, LOG2L>(r3, im3, lrj, lij, 0, 1, 0, t, tw3, act);
            }
            if (act && row0 + rl < a.rows) {
                const int64_t row = row0 + rl;
                // slots w < W - c take mode w (zero when w > c); slots w >= W - c
                // take mode L - W + w
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int kx = R * (t + e * Tn) + q;
                    C v;
                    v.x = r3[0][e];
                    v.y = im3[0][e];
                    if (kx < W - c) {
                        if (kx > c) { v.x = 0; v.y = 0; }
                        Zo[zat(pl, row, kx)] = v;
                    } else if (kx >= L - c) {
                        Zo[zat(pl, row, W - L + kx)] = v;
                    }
                }
            }
        }
    }

    if (MODE == FM_VKEY || MODE == FM_RELAX || (flags & (RF_PROJECT | RF_TRACK))) {
        // counts of the workgroup: packed 21 bits each (at most 2048 per workgroup)
        unsigned long long packed = wave_sum(nflip | (nfb << 21) | (nbad << 42));
        unsigned long long dbits = (unsigned long long)__double_as_longlong(dmax);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long ob = (unsigned long long)__shfl_xor((long long)dbits, o, 64);
            dbits = ob > dbits ? ob : dbits;
        }
        if ((tid & 63) == 0) {
            if (packed) atomicAdd(&wg_cnt[0], packed);
            if (dbits) atomicMax(&wg_cnt[1], dbits);
        }
        __syncthreads();
        if (tid == 0) {
            // the workgroup's packed counts into its own slot (summed per
            // iteration after the loop: no same-address atomics from every
            // workgroup at the end of the pass); the largest change by atomic max
            if (a.cnt_part)
                a.cnt_part[((int64_t)b * a.K + (a.iter - 1)) * gridDim.x + blockIdx.x] = wg_cnt[0];
            if ((flags & RF_TRACK) && a.delta_bits && wg_cnt[1])
                atomicMax(a.delta_bits + (int64_t)b * a.K + (a.iter - 1), wg_cnt[1]);
        }
    }
}

template <typename T, int n, int LOG2L, bool PM>
__global__ void __launch_bounds__((RowFastShape<T, n, LOG2L>::THREADS), (RowFastShape<T, n, LOG2L>::WAVES))
    row_fast(const FastRowArgs a)
{
    row_fast_body<T, n, LOG2L, PM, FM_ITER>(a, blockIdx.x);
}

template <typename T, int n, int LOG2L>
__global__ void __launch_bounds__((RowFastShape<T, n, LOG2L>::THREADS), (RowFastShape<T, n, LOG2L>::WAVES))
    row_fast_vjp(const FastRowArgs a)
{
    row_fast_body<T, n, LOG2L, false, FM_VJP>(a, blockIdx.x);
}

template <typename T, int n, int LOG2L>
__global__ void __launch_bounds__((RowFastShape<T, n, LOG2L>::THREADS), (RowFastShape<T, n, LOG2L>::WAVES))
    row_fast_relax(const FastRowArgs a)
{
    row_fast_body<T, n, LOG2L, false, FM_RELAX>(a, blockIdx.x);
}

// n = 4: the Jacobi of every point with its singular values takes more than 128
// registers; one workgroup per CU without scratch memory (whose set-up delays
// the start of the workgroups) rather than two with it: 256^2 in float, six
// steps 596 -> 571 us.
template <typename T, int n, int LOG2L>
__global__ void __launch_bounds__((RowFastShape<T, n, LOG2L>::THREADS),
                                  (n == 4 ? (RowFastShape<T, n, LOG2L>::THREADS + 255) / 256
                                          : RowFastShape<T, n, LOG2L>::WAVES))
    row_fast_vkey(const FastRowArgs a)
{
    row_fast_body<T, n, LOG2L, false, FM_VKEY>(a, blockIdx.x);
}

// ---------------------------------------------------------------------------
// The points that the volume-preserving selection puts on the other side
// ---------------------------------------------------------------------------
// One workgroup per row_fast workgroup (at least 512 points, whole rows).  A
// point whose membership differs from the sign of its Delta E changes from Q to
// the candidate of the other determinant (Lemma 7.1, vp_change), in the field and in
// the row spectra that row_fast_vkey wrote.  Once the volume has settled few do: the
// selection moves the cut only as far as the volume drifted in one step, and the change
// is added to their rows' spectra by direct sums over the kept modes.  A workgroup with
// more than VFIX_DIRECT of them (rough data) lists itself for volume_redo, which
// transforms those rows again.  Rows without such points end after reading Delta E and
// the det signs.
// Bound by its chain of memory round trips (flags, point, spectra), not by the 300 to
// 660 points in 140 to 230 rows that it treats at 512^2, n = 3 in float: 8.5 us, and 4 for
// the empty volume_redo (13 with the points read back from the spectra).  A step of
// 2048^2, n = 3, from a field with 30 % of the points flipped, all of which change side:
// 0.74 ms; with direct sums for each of them 6.2, by the general passes 1.23.
// Dynamic LDS: the twiddle table.
constexpr int VFIX_NT = 512;
constexpr int VFIX_DIRECT = 64;

template <typename T, int n>
__global__ void __launch_bounds__(VFIX_NT, 4) volume_fix(const VolFixArgs f)
{
    constexpr int NN = n * n, PL = (NN + 1) / 2, NT = VFIX_NT, PER = 2048 / NT;
    typedef typename cx<T>::type C;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* twl = reinterpret_cast<C*>(smem_raw);
    const FastRowArgs& a = f.r;
    __shared__ unsigned short list[2048];
    __shared__ int wcnt[PER][NT / 64];
    __shared__ T delta[VFIX_DIRECT][2 * PL];
    __shared__ unsigned wflip[NT / 64];
    const int b = blockIdx.y, tid = threadIdx.x, L = a.L, W = a.W, c = a.band;
    const int lg = 31 - __clz(L), rpw = L >= 512 ? 1 : 512 >> lg;
    const int64_t row0 = (int64_t)blockIdx.x * rpw;
    const int64_t p0 = row0 * L;
    const int64_t left = a.npts - p0;
    const int P = (int)(left < (int64_t)rpw * L ? left : (int64_t)rpw * L);  // points of this workgroup, <= 2048
    const T* vde = reinterpret_cast<const T*>(a.vde) + (size_t)b * a.npts + p0;
    int8_t* sgn = a.sgn + (size_t)b * a.npts + p0;
    T de[PER];
    int8_t old[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = k * NT + tid;
        de[k] = i < P ? vde[i] : (T)0;
        old[k] = i < P ? sgn[i] : (int8_t)0;
    }
    const VpSel sel = f.vsel[b];
    // the changed points, listed in index order
    unsigned flips = 0, chg = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (k * NT >= P) continue;  // uniform
        const int i = k * NT + tid;
        bool ch = false;
        if (i < P) {
            const bool in = vp_member(sel, vp_key(de[k]), p0 + i);
            ch = in == (bool)__builtin_signbit(de[k]);
            const int8_t now = in ? 1 : -1;
            if (old[k] != now) {
                sgn[i] = now;
                ++flips;
            }
        }
        chg |= ch ? 1u << k : 0u;
        const unsigned long long bal = __ballot(ch);
        if ((tid & 63) == 0) wcnt[k][tid >> 6] = __popcll(bal);
    }
    flips = (unsigned)wave_sum((unsigned long long)flips);
    if ((tid & 63) == 0) wflip[tid >> 6] = flips;
    __syncthreads();
    int m = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (k * NT >= P) continue;
        const unsigned long long bal = __ballot((chg >> k) & 1u);
        int at = m;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) {
            at += w < (tid >> 6) ? wcnt[k][w] : 0;
            m += wcnt[k][w];
        }
        at += __popcll(bal & ((1ull << (tid & 63)) - 1ull));
        if ((chg >> k) & 1u) list[at] = (unsigned short)(k * NT + tid);
    }
    if (tid == 0 && a.cnt_part) {
        unsigned all = 0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) all += wflip[w];
        if (all) a.cnt_part[((int64_t)b * a.K + (a.iter - 1)) * gridDim.x + blockIdx.x] += all;
    }
    if (m == 0) return;  // uniform
    const bool forward = (a.flags & RF_FORWARD) != 0, direct = forward && m <= VFIX_DIRECT;
    if (forward && !direct && tid == 0)
        f.redo[(size_t)b * gridDim.x + atomicAdd(f.nredo + b, 1u)] = blockIdx.x;
    if (direct)
        for (int i = tid; i < L; i += NT) twl[i] = reinterpret_cast<const C*>(a.tw)[i];
    __syncthreads();  // the list is written
    T* Aout = reinterpret_cast<T*>(a.slot ? *a.slot : a.Aout) + field_base(a.foff, b, NN * a.npts) + p0;
    const T* vdir = reinterpret_cast<const T*>(a.vdir) + (size_t)b * n * a.npts + p0;
    for (int j = tid; j < m; j += NT) {
        const int i = list[j];
        T q[NN], v[n], d[NN];
#pragma unroll
        for (int k = 0; k < NN; ++k) q[k] = Aout[(int64_t)k * a.npts + i];
#pragma unroll
        for (int k = 0; k < n; ++k) v[k] = n > 1 ? vdir[(int64_t)k * a.npts + i] : (T)0;
        vp_change<T, n>(!(bool)__builtin_signbit(vde[i]), v, q, d);
#pragma unroll
        for (int k = 0; k < NN; ++k) Aout[(int64_t)k * a.npts + i] = q[k];
        if (direct) {
#pragma unroll
            for (int k = 0; k < NN; ++k) delta[j][k] = d[k];
            if (NN & 1) delta[j][NN] = (T)0;
        }
    }
    if (!direct) return;
    __syncthreads();
    // a thread owns its (plane, mode) pairs, the points of a row follow each other in
    // the list
    C* Zo = reinterpret_cast<C*>(a.Zout) + (size_t)b * PL * a.rows * W;
    for (int e = tid; e < PL * W; e += NT) {
        const int p = e / W, w = e - p * W;
        if (W != L && w > c && w < W - c) continue;  // unused slot: stays zero
        const int kx = (W == L || w <= c) ? w : L - W + w;
        int j = 0;
        while (j < m) {
            const int r = list[j] >> lg;
            C* z = &Zo[((size_t)p * a.rows + row0 + r) * W + w];
            C v = *z;
            int j1 = j;
            while (j1 < m && list[j1] >> lg == r) ++j1;
#pragma unroll 4
            for (; j < j1; ++j) {
                const C t = twl[(kx * (list[j] & (L - 1))) & (L - 1)];
                const T dr = delta[j][2 * p], di = delta[j][2 * p + 1];
                v.x += dr * t.x - di * t.y;  // (dr + i di) exp(-2 pi i kx x / L)
                v.y += dr * t.y + di * t.x;
            }
            *z = v;
        }
    }
}

// The rows that volume_fix listed: their spectra from the field again.  As a rule the
// list is empty and the workgroups end at once.
template <typename T, int n, int LOG2L>
__global__ void __launch_bounds__((RowFastShape<T, n, LOG2L>::THREADS)) volume_redo(const VolFixArgs f)
{
    const unsigned m = f.nredo[blockIdx.y];
    for (unsigned i = blockIdx.x; i < m; i += gridDim.x) {
        row_fast_body<T, n, LOG2L, false, FM_REDO>(f.r, f.redo[(size_t)blockIdx.y * f.groups + i]);
        __syncthreads();  // the lines in LDS have been read
    }
}

// ---------------------------------------------------------------------------
// Column pass over the stored columns
// ---------------------------------------------------------------------------

// Dynamic LDS of a heat_fast workgroup: the TX padded lines, then the twiddle
// table when it fits.
template <typename T, int LOG2L, int TX>
struct HeatFastShape {
    static constexpr int L = 1 << LOG2L;
    static constexpr size_t LINES = (size_t)TX * (L + L / 8) * 2 * sizeof(T);
    static constexpr size_t TW_BYTES = (size_t)L * 2 * sizeof(T);
    static constexpr bool TW_LDS = LINES + TW_BYTES <= 159744;
    static constexpr size_t LDS = LINES + (TW_LDS ? TW_BYTES : 0);
};

template <typename T, int LOG2L, int TX, int MODE>
__device__ __forceinline__ void heat_fast_body(const FastColArgs& a)
{
    typedef typename cx<T>::type C;
    typedef FftShape<LOG2L> F;
    constexpr int L = F::L, Tn = F::Tn;
    constexpr int LP = L + L / 8;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* lr = reinterpret_cast<T*>(smem_raw);
    T* li = lr + (size_t)TX * LP;

    const int b = blockIdx.y;
    const int tid = threadIdx.x;
    const int cc = tid % TX, t = tid / TX;
    // XCD-aware order: the eight XCDs (own L2 each) get contiguous runs of tiles
    const int64_t nwgx = gridDim.x;
    const int64_t wg = ((nwgx & 7) || !a.xcd_remap) ? (int64_t)blockIdx.x
                                                    : (int64_t)(blockIdx.x & 7) * (nwgx >> 3) + (blockIdx.x >> 3);
    const int64_t o = wg / a.tiles;
    const int col = (int)(wg - o * a.tiles) * TX + cc;
    C* Zc = reinterpret_cast<C*>(a.Z) + (size_t)b * a.field_elems + o * (int64_t)L * a.W + col;
    // every independent global load first (column data, symbol, twiddles, the
    // stop marks): at the start of a launch each round trip is a cold miss
    T r[1][8], im[1][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const C v = Zc[(int64_t)(t + e * Tn) * a.W];
        r[0][e] = v.x;
        im[0][e] = v.y;
    }
    const T* lrow = reinterpret_cast<const T*>(a.lam_row) + b * a.lam_row_stride;
    const T lcol = reinterpret_cast<const T*>(a.lam_col)[b * a.lam_col_stride + col];
    T lam[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) lam[e] = lrow[t + e * Tn];
    // the twiddle table staged in LDS after the tile's lines where it fits:
    // 8/TX loads per thread instead of 7 per radix-8 stage
    const C* twg = reinterpret_cast<const C*>(a.tw);
    C* twl = reinterpret_cast<C*>(li + (size_t)TX * LP);
    if constexpr (HeatFastShape<T, LOG2L, TX>::TW_LDS) {
#pragma unroll
        for (int m = tid; m < L; m += TX * Tn) twl[m] = twg[m];
        __syncthreads();
    }
    Twiddles<T, LOG2L> tw;
    load_twiddles<T, LOG2L>(tw, HeatFastShape<T, LOG2L, TX>::TW_LDS ? twl : twg, t);
    const bool marks = a.iter > 0 && a.stop_iter;
    const int stop = marks ? a.stop_iter[b] : a.iter;
    const bool check_tol = marks && a.delta_bits && a.tol > 0.0 && a.iter >= 2;
    const unsigned long long dbits = check_tol ? a.delta_bits[(int64_t)b * a.K + (a.iter - 2)] : 0ull;
    if (marks) {
        if (stop < a.iter) return;  // uniform per workgroup
        // the first pass of iteration s stops field b when s-1 changed it by <= tol
        if (check_tol && __longlong_as_double((long long)dbits) <= a.tol) {
            if (blockIdx.x == 0 && tid == 0) atomicMin(a.stop_iter + b, a.iter - 1);
            return;
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if constexpr (MODE == HF_RESOLVENT) lam[e] = (T)a.rnorm / ((T)1 - (T)a.rdt * (lam[e] + lcol));
        else lam[e] *= lcol;
    }
    fft_lines<T, -1, 1, LOG2L>(r, im, lr, li, 0, TX, cc, t, tw);
    if (a.epart) {
        // this thread's eight terms in the plan's precision (a.wide: in double), the
        // wave's sum in double
        double part;
        if (sizeof(T) == 4 && a.wide) {
            part = 0.0;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                part += (double)lam[e] * ((double)r[0][e] * (double)r[0][e] + (double)im[0][e] * (double)im[0][e]);
        } else {
            T acc = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc += lam[e] * (r[0][e] * r[0][e] + im[0][e] * im[0][e]);
            part = (double)acc;
        }
        const double s = wave_sum(part);
        const int slot = a.slot >= 0 ? a.slot : a.stop_iter[b];
        if ((tid & 63) == 0)
            a.epart[((int64_t)b * (a.K + 1) + slot) * a.nwg + wg * (blockDim.x >> 6) + (tid >> 6)] = s;
    }
    if constexpr (MODE == HF_SAVE || MODE == HF_DOT || MODE == HF_DTAU) {
        // a thread's eight values side by side: the two passes run the same
        // launch shape, so the layout of a.spec is their own
        C* S = reinterpret_cast<C*>(a.spec) + ((size_t)b * gridDim.x + wg) * (size_t)(TX * L) + tid;
        if (MODE == HF_SAVE || (MODE == HF_DTAU && a.spec)) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                C v;
                v.x = r[0][e];
                v.y = im[0][e];
                S[e * (TX * Tn)] = v;
            }
        }
        if constexpr (MODE == HF_DOT || MODE == HF_DTAU) {
            const T kx = (T)(a.W == a.N1 ? (2 * col < a.N1 ? col : col - a.N1) : (col <= a.band ? col : col - a.W));
            double acc = 0.0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int m = t + e * Tn;
                const T ky = (T)(2 * m < L ? m : m - L);
                const T mu = lam[e] * ((T)-39.478417604357434475337963999505 * (kx * kx + ky * ky));  // -4 pi^2 |k|^2
                if constexpr (MODE == HF_DTAU) {
                    lam[e] = mu;
                } else {
                    const C v = S[e * (TX * Tn)];
                    acc += (double)mu * ((double)r[0][e] * (double)v.x + (double)im[0][e] * (double)v.y);
                }
            }
            if constexpr (MODE == HF_DOT) {
                const double s = wave_sum(acc);
                if ((tid & 63) == 0) a.dpart[(int64_t)b * a.nwg + wg * (blockDim.x >> 6) + (tid >> 6)] = s;
            }
        }
    }
    if (!a.apply) return;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        r[0][e] *= lam[e];
        im[0][e] *= lam[e];
    }
    fft_lines<T, +1, 1, LOG2L>(r, im, lr, li, 0, TX, cc, t, tw);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        C v;
        v.x = r[0][e];
        v.y = im[0][e];
        Zc[(int64_t)(t + e * Tn) * a.W] = v;
    }
}

template <typename T, int LOG2L, int TX>
__global__ void __launch_bounds__(TX * (1 << LOG2L) / 8) heat_fast(const FastColArgs a)
{
    heat_fast_body<T, LOG2L, TX, HF_PLAIN>(a);
}

template <typename T, int LOG2L, int TX, int MODE>
__global__ void __launch_bounds__(TX * (1 << LOG2L) / 8) heat_fast_adj(const FastColArgs a)
{
    heat_fast_body<T, LOG2L, TX, MODE>(a);
}

// ---------------------------------------------------------------------------
// Plane pass of the 3-D iteration: the heat step along y and z
// ---------------------------------------------------------------------------

// The N0 x N1 plane of one packed plane and stored x mode w, contiguous in
// Z[plane][w][z][y] as the row pass stores it for 3-D, is loaded once,
// transformed along y and then z in LDS, its Lyapunov partial taken, multiplied
// by lambda_z(kz) lambda_y(ky) lambda_x(w), transformed back along z and y, and
// stored in place: the whole diffusion between two row passes in one read and
// one write of the spectra.  Each thread holds two lines of eight values.  The
// plane sits in LDS as complex pairs (real and imaginary part side by side: one
// address per element) in rows of odd pitch, so that the z lines spread over the
// banks; the exchanges inside a line use the XOR-permuted positions of
// line_index<LIX_XOR>.  One workgroup per plane, or as many planes as fill a
// wave where a plane has fewer than 1024 points (a wider workgroup of small
// planes would leave CUs idle: 16 x 16 x 128 has a few hundred planes).
// Bound by memory where the spectra are large (128^3 in float, n = 3: 53 us,
// 2.8 TB/s), by the latency of its chain of transforms where they are not.
template <typename T, int LOG2Y, int LOG2Z>
struct PlaneFastShape {
    static constexpr int NY = 1 << LOG2Y, NZ = 1 << LOG2Z;
    static constexpr int TY = NY / 8, TZ = NZ / 8;
    static constexpr int PT = NY * NZ / 16;         // threads of one plane
    static constexpr int G = PT < 64 ? 64 / PT : 1; // planes per workgroup
    static constexpr int THREADS = G * PT;
    static constexpr int PZ = NY + 1;  // row pitch in complex elements
    // the planes, then the y and z twiddle tables
    static constexpr size_t LDS = ((size_t)G * NZ * PZ + NY + NZ) * 2 * sizeof(T);
};

template <typename T, int LOG2Y, int LOG2Z>
__global__ void __launch_bounds__((PlaneFastShape<T, LOG2Y, LOG2Z>::THREADS)) plane_fast(const FastColArgs a)
{
    typedef PlaneFastShape<T, LOG2Y, LOG2Z> S;
    typedef typename cx<T>::type C;
    constexpr int NY = S::NY, NZ = S::NZ, TY = S::TY, TZ = S::TZ, PZ = S::PZ;
    extern __shared__ __align__(16) unsigned char smem_raw[];

    const int b = blockIdx.y;
    const int tid = threadIdx.x % S::PT;
    const int pw = threadIdx.x / S::PT;  // this plane among the workgroup's
    // element o of the plane: lc[2 o] (real), lc[2 o + 1] (imaginary)
    T* lc = reinterpret_cast<T*>(smem_raw) + (S::G > 1 ? 2 * pw * NZ * PZ : 0);
    // packed plane * W + stored mode; the last workgroup's planes beyond the
    // field's read its last one and store nothing
    const int64_t nplanes = a.field_elems / (NZ * NY);
    const bool live = S::G == 1 || (int64_t)blockIdx.x * S::G + pw < nplanes;
    const int64_t wg = live ? (int64_t)blockIdx.x * S::G + pw : nplanes - 1;
    const int w = (int)(wg % a.W);
    C* Zp = reinterpret_cast<C*>(a.Z) + (size_t)b * a.field_elems + (size_t)wg * NZ * NY;
    // y lines: group gy takes z = gy and gy + NZ/2, lane ty elements y = ty + e TY
    const int gy = tid / TY, ty = tid - gy * TY;
    T r[2][8], im[2][8];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const C v = Zp[(gy + h * (NZ / 2)) * NY + ty + e * TY];
            r[h][e] = v.x;
            im[h][e] = v.y;
        }
    // z lines: group gz takes ky = gz and gz + NY/2, lane tz elements kz = tz + e TZ
    const int gz = tid / TZ, tz = tid - gz * TZ;
    const T* lz = reinterpret_cast<const T*>(a.lam_row) + b * a.lam_row_stride;
    const T* ly = reinterpret_cast<const T*>(a.lam_y) + b * a.lam_y_stride;
    const T lx = reinterpret_cast<const T*>(a.lam_col)[b * a.lam_col_stride + w];
    // twiddles are read stage by stage from copies of the tables in LDS (the
    // copies of global reads would be merged across the kernel and kept in
    // registers, more than the 1024-thread instance's 128 hold), and the symbol
    // where it is used
    C* twl = reinterpret_cast<C*>(smem_raw) + (size_t)S::G * NZ * PZ;
    for (int m = threadIdx.x; m < NY + NZ; m += S::THREADS)
        twl[m] = m < NY ? reinterpret_cast<const C*>(a.tw_y)[m] : reinterpret_cast<const C*>(a.tw)[m - NY];
    __syncthreads();
    const TwiddleTable<T, LOG2Y> twy{twl};
    const TwiddleTable<T, LOG2Z> twz{twl + NY};
    const bool marks = a.iter > 0 && a.stop_iter;
    const int stop = marks ? a.stop_iter[b] : a.iter;
    const bool check_tol = marks && a.delta_bits && a.tol > 0.0 && a.iter >= 2;
    const unsigned long long dbits = check_tol ? a.delta_bits[(int64_t)b * a.K + (a.iter - 2)] : 0ull;
    if (marks) {
        if (stop < a.iter) return;  // uniform per workgroup
        // the first pass of iteration s stops field b when s-1 changed it by <= tol
        if (check_tol && __longlong_as_double((long long)dbits) <= a.tol) {
            if (blockIdx.x == 0 && threadIdx.x == 0) atomicMin(a.stop_iter + b, a.iter - 1);
            return;
        }
    }
    // A lane index the compiler takes as a new value: the index arithmetic of
    // one transform is then not kept in registers for the transform back.
    auto fresh = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    // y line h of the group: element y at 2 ((gy + h NZ/2) PZ + y); z line h:
    // element z at 2 (z PZ + gz + h NY/2)
    const int yl = 2 * gy * PZ, yp = 2 * (NZ / 2) * PZ;
    const int zl = 2 * gz, zp = 2 * (NY / 2);

    // forward along y (rows z of the plane), the result to LDS
    fft_lines<T, -1, 2, LOG2Y, LIX_XOR>(r, im, lc, lc + 1, yp, 2, yl, fresh(ty), twy);
    __syncthreads();  // the rows' last exchanges have been read
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int o = yl + h * yp + 2 * (ty + e * TY);
            lc[o] = r[h][e];
            lc[o + 1] = im[h][e];
        }
    __syncthreads();
    // forward along z (columns ky)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int o = zl + h * zp + 2 * PZ * (tz + e * TZ);
            r[h][e] = lc[o];
            im[h][e] = lc[o + 1];
        }
    fft_lines<T, -1, 2, LOG2Z, LIX_XOR>(r, im, lc, lc + 1, zp, 2 * PZ, zl, fresh(tz), twz);
    T lzv[8], lyv[2];
#pragma unroll
    for (int e = 0; e < 8; ++e) lzv[e] = lz[tz + e * TZ] * lx;
#pragma unroll
    for (int h = 0; h < 2; ++h) lyv[h] = ly[gz + h * (NY / 2)];
    if (a.epart) {
        // this thread's terms in the plan's precision, the wave's sum in double
        T acc = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc += (lzv[e] * lyv[h]) * (r[h][e] * r[h][e] + im[h][e] * im[h][e]);
        const double sum = wave_sum(live ? (double)acc : 0.0);
        const int slot = a.slot >= 0 ? a.slot : a.stop_iter[b];
        if ((threadIdx.x & 63) == 0)
            a.epart[((int64_t)b * (a.K + 1) + slot) * a.nwg + (int64_t)blockIdx.x * (S::THREADS >> 6) +
                    (threadIdx.x >> 6)] = sum;
    }
    if (!a.apply) return;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const T lm = lzv[e] * lyv[h];
            r[h][e] *= lm;
            im[h][e] *= lm;
        }
    // back along z, then y
    fft_lines<T, +1, 2, LOG2Z, LIX_XOR>(r, im, lc, lc + 1, zp, 2 * PZ, zl, fresh(tz), twz);
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int o = zl + h * zp + 2 * PZ * (tz + e * TZ);
            lc[o] = r[h][e];
            lc[o + 1] = im[h][e];
        }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int o = yl + h * yp + 2 * (ty + e * TY);
            r[h][e] = lc[o];
            im[h][e] = lc[o + 1];
        }
    fft_lines<T, +1, 2, LOG2Y, LIX_XOR>(r, im, lc, lc + 1, yp, 2, yl, fresh(ty), twy);
    if (!live) return;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            C v;
            v.x = r[h][e];
            v.y = im[h][e];
            Zp[(gy + h * (NZ / 2)) * NY + ty + e * TY] = v;
        }
}

}  // namespace mbo

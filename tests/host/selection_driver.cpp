// The three-launch selection (mbo_volume.hip, launch_select_list) on the CPU against a
// sort: spread, clustered, equal, nearly equal and non-finite values, one to three
// fields, every kind of rank; twice on the same buffers, which it has to leave at zero.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <numeric>
#include <random>
#include <vector>

#include "mbo_internal.hpp"

using namespace mbo;

// launchers that the selection's source names and this program does not reach
namespace mbo {
hipError_t launch_fill_u64(unsigned long long*, int64_t, unsigned long long, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_row_vp_f32(int, int, const RowArgs&, dim3, dim3, size_t, hipStream_t, bool) { return hipErrorUnknown; }
hipError_t launch_row_vp_f64(int, int, const RowArgs&, dim3, dim3, size_t, hipStream_t, bool) { return hipErrorUnknown; }
}  // namespace mbo

static unsigned long long key(float v)
{
    unsigned u;
    std::memcpy(&u, &v, sizeof u);
    if ((u << 1) == 0u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

static unsigned long long key(double v)
{
    unsigned long long u;
    std::memcpy(&u, &v, sizeof u);
    if ((u << 1) == 0ull) u = 0ull;
    return (u >> 63) ? ~u : (u | (1ull << 63));
}

static const int KINDS = 9;

static double value(int kind, std::mt19937& g)
{
    const double x = std::normal_distribution<double>()(g);
    const unsigned r = (unsigned)g();
    switch (kind) {
    case 1: return 0.8 + 0.05 * x;
    case 2: return 1.0;
    case 3: return 1.0 + 1e-7 * x;
    case 4: return (double)(r % 3) - 1.0;
    case 5: return (r & 1) ? 0.0 : -0.0;
    case 6: return 1.5 + 1e-15 * (r % 50);
    case 7: return x * std::pow(10.0, (int)(r % 30) - 20);
    case 8: return r % 100 == 0 ? INFINITY : r % 100 == 1 ? -INFINITY : r % 200 == 7 ? NAN : -0.3 + 1e-9 * x;
    }
    return x;
}

static bool member(const VpSel& s, unsigned long long k, int64_t i)
{
    if (s.mode == VS_ALL) return true;
    if (s.mode == VS_TIES_ALL) return k >= s.kstar;
    if (s.mode == VS_TIES_PART) return k > s.kstar || (k == s.kstar && i <= s.istar);
    return false;
}

template <typename T>
static bool round(std::mt19937& g, int it)
{
    // below, at and above the 8192 points that one workgroup takes
    static const int sizes[] = {512, 4096, 8192, 8704, 16384, 20480, 32768};
    const int B = 1 + (int)(g() % 3);
    const int64_t np = sizes[g() % 7], chunks = (np + SEL_CHUNK - 1) / SEL_CHUNK;
    std::vector<T> v((size_t)(B * np));
    std::vector<int64_t> n_plus((size_t)B);
    for (int b = 0; b < B; ++b) {
        const int kind = (int)(g() % KINDS);
        for (int64_t i = 0; i < np; ++i) v[(size_t)(b * np + i)] = (T)value(kind, g);
        const int64_t ranks[8] = {0, np, 1, np - 1, (int64_t)(g() % np), (int64_t)(g() % np), np / 2, (int64_t)(g() % np)};
        n_plus[(size_t)b] = ranks[g() % 8];
    }
    const size_t sb = (size_t)B, sp = (size_t)(B * np);
    std::vector<VpSel> st(sb);
    std::vector<unsigned> hist(sb << SEL_BITS), tcnt(sb * (size_t)chunks), done(sb), count(sb), hist2(sb * SEL_HIST2),
        over(sb, 77u), clear(sb, 99u), idx(sp);
    std::vector<unsigned long long> keys(sp);
    SelListArgs a;
    std::memset(&a, 0, sizeof a);
    a.s.dE = v.data();
    a.s.npts = np;
    a.s.nplus = n_plus.data();
    a.s.st = st.data();
    a.s.hist = hist.data();
    a.s.tcnt = tcnt.data();
    a.s.chunks = chunks;
    a.s.done = done.data();
    a.key = keys.data();
    a.idx = idx.data();
    a.count = count.data();
    a.hist2 = hist2.data();
    a.over = over.data();
    a.clear = clear.data();
    auto zero = [](const std::vector<unsigned>& x) {
        return std::all_of(x.begin(), x.end(), [](unsigned u) { return u == 0u; });
    };
    for (int rep = 0; rep < 2; ++rep) {
        if (launch_select_list(sizeof(T) == 8 ? 0 : 1, a, B, nullptr) != hipSuccess) return false;
        for (int b = 0; b < B; ++b) {
            const T* x = v.data() + (size_t)(b * np);
            std::vector<int> o((size_t)np);
            std::iota(o.begin(), o.end(), 0);
            std::stable_sort(o.begin(), o.end(), [&](int i, int j) { return key(x[i]) > key(x[j]); });
            for (int64_t r = 0; r < np; ++r)
                if (member(st[(size_t)b], key(x[o[(size_t)r]]), o[(size_t)r]) != (r < n_plus[(size_t)b])) {
                    std::printf("round %d, field %d of %d, %lld points, n_plus %lld: wrong at rank %lld\n", it, b, B,
                                (long long)np, (long long)n_plus[(size_t)b], (long long)r);
                    return false;
                }
        }
        if (!zero(hist) || !zero(hist2) || !zero(count) || !zero(done) || !zero(clear)) {
            std::printf("round %d: buffers not left at zero\n", it);
            return false;
        }
    }
    return true;
}

int main(int argc, char** argv)
{
    std::mt19937 g((unsigned)std::atoi(argv[1]));
    bool ok = argc == 3;
    for (int i = 0; ok && i < std::atoi(argv[2]); ++i) ok = (i & 1) ? round<float>(g, i) : round<double>(g, i);
    if (ok) std::printf("ok\n");
    return ok ? 0 : 1;
}

// Host side of plans under refused allocations and changed streams (fake_runtime.hpp).
// Each scenario prints "ok" or what went wrong; run by tests/test_host_runtime.py.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <thread>
#include <vector>

#include "fake_runtime.hpp"
#include "mbo.h"

static int bad = 0;
#define CHECK(x)                                                      \
    do {                                                              \
        if (!(x)) {                                                   \
            std::printf("line %d: %s fails\n", __LINE__, #x);         \
            bad = 1;                                                  \
        }                                                             \
    } while (0)

// The symbol that the column (or plane) pass was launched with is that of tau, in double.
static bool symbol_is(double tau, int64_t N1)
{
    const double* lam = static_cast<const double*>(fake::heat.lam_col);
    if (!lam) return false;
    const double pi = 3.14159265358979323846;
    for (int k = 0; k < 3; ++k)
        if (std::fabs(lam[k] * (double)N1 - std::exp(-4.0 * pi * pi * tau * k * k)) > 1e-12) return false;
    return true;
}

// mbo_plan_set_tau and mbo_plan_set_path whose tables are refused leave the plan as it
// was, and the same call again changes it.
static void set_tau(int d)
{
    const int64_t N[3] = {64, 64, 64};
    mbo_plan_t p = nullptr;
    CHECK(mbo_plan(&p, d, N, 2, 1, 1e-3, MBO_F64, 0.0, nullptr) == MBO_OK);
    if (!p) return;
    std::vector<double> A((size_t)4 * 64 * 64 * (d == 3 ? 64 : 1), 1.0), B(A.size());
    auto diffused = [&](double tau) {
        std::memset(&fake::heat, 0, sizeof fake::heat);
        return mbo_diffuse(p, A.data(), B.data()) == MBO_OK && symbol_is(tau, 64);
    };
    CHECK(diffused(1e-3));
    for (int k = 1; k <= 3; ++k) {  // whichever allocation is refused
        fake::fail_in = k;
        const mbo_status s = mbo_plan_set_tau(p, 2e-3);
        const bool refused = fake::fail_in == 0;
        fake::fail_in = 0;
        CHECK(!refused || s != MBO_OK);
        CHECK(s == MBO_OK || diffused(1e-3));
        CHECK(mbo_plan_set_tau(p, 2e-3) == MBO_OK);
        CHECK(diffused(2e-3));
        CHECK(mbo_plan_set_tau(p, 1e-3) == MBO_OK);
        CHECK(diffused(1e-3));
    }
    CHECK(mbo_plan_set_path(p, MBO_PATH_GENERIC) == MBO_OK);
    int path = -1, c = 0, w = 0;
    fake::fail_in = 1;
    CHECK(mbo_plan_set_path(p, MBO_PATH_FULL) != MBO_OK);
    fake::fail_in = 0;
    CHECK(mbo_plan_path(p, 0, &path, &c, &w) == MBO_OK && path == MBO_PATH_GENERIC);
    fake::reset();
    CHECK(mbo_diffuse(p, A.data(), B.data()) == MBO_OK && fake::count("row_fast") == 0);
    CHECK(mbo_plan_set_path(p, MBO_PATH_BANDED) == MBO_OK);
    CHECK(diffused(1e-3));
    CHECK(mbo_plan_destroy(p) == MBO_OK);
    CHECK(fake::held == 0);
}

// The band-limited volume-preserving iteration takes workspace that the general passes
// do without: where it is refused the call runs those, and the next call tries again.
static void volume_memory()
{
    const int64_t N[2] = {64, 64};
    mbo_plan_t p = nullptr;
    CHECK(mbo_plan(&p, 2, N, 3, 2, 1e-3, MBO_F32, 0.0, nullptr) == MBO_OK);
    if (!p) return;
    std::vector<float> A((size_t)2 * 9 * 64 * 64, 1.0f);
    std::vector<double> E((size_t)2 * 4);
    int64_t used[2];
    for (int round = 0; round < 2; ++round) {
        fake::reset();
        fake::fail_above = 150000;  // the spectra take more, Delta E (32 KB) and the logs less
        CHECK(mbo_iterate_volume(p, A.data(), 3, nullptr, used, E.data(), nullptr, nullptr) == MBO_OK);
        CHECK(fake::count("row_fast_vkey") == 0 && fake::count("volume_fix") == 0);
        CHECK(fake::count("row_vp") == (round == 0 ? 6 : 0));  // the captured call is kept
        CHECK(fake::count("graph") == 1);
    }
    fake::fail_above = 0;
    fake::reset();
    CHECK(mbo_iterate_volume(p, A.data(), 3, nullptr, used, E.data(), nullptr, nullptr) == MBO_OK);
    CHECK(fake::count("row_fast_vkey") == 3 && fake::count("volume_fix") == 3 && fake::count("row_vp") == 0);
    CHECK(mbo_plan_destroy(p) == MBO_OK);
    CHECK(fake::held == 0);
}

// The same of the adjoint's calls.
static void adjoint_memory()
{
    const int64_t N[2] = {64, 64};
    for (int n = 2; n <= 4; ++n) {
        mbo_plan_t p = nullptr;
        CHECK(mbo_plan(&p, 2, N, n, 1, 1e-3, MBO_F64, 0.0, nullptr) == MBO_OK);
        if (!p) return;
        CHECK(mbo_plan_set_path(p, MBO_PATH_FULL) == MBO_OK);  // spectra larger than a field
        std::vector<double> A((size_t)n * n * 64 * 64, 1.0), G(A.size()), O(A.size());
        double dtau = 0.0, dot = 0.0;
        const size_t field = A.size() * 8, spec = (size_t)(n * n + 1) / 2 * 64 * 64 * 16;
        fake::fail_above = n == 3 ? field : spec - 1;  // n = 2, 4: as large as a field
        fake::reset();
        CHECK(mbo_diffuse_dtau(p, A.data(), O.data(), G.data(), &dot) == MBO_OK);
        CHECK(fake::count("heat_fast_adj") == 0 && fake::count("col") == 1);
        if (n == 3) {
            CHECK(mbo_step_vjp(p, A.data(), G.data(), &dtau) == MBO_OK);
            CHECK(fake::count("heat_fast_adj") == 0 && fake::count("vjp") == 1);
        } else {
            CHECK(mbo_step_vjp(p, A.data(), G.data(), &dtau) == MBO_ERR_ALLOC);  // the general passes need two fields
        }
        fake::fail_above = 0;
        fake::reset();
        CHECK(mbo_step_vjp(p, A.data(), G.data(), &dtau) == MBO_OK);
        CHECK(mbo_diffuse_dtau(p, A.data(), O.data(), G.data(), &dot) == MBO_OK);
        CHECK(fake::count("heat_fast_adj") > 0 && fake::count("col") == 0);
        CHECK(mbo_plan_destroy(p) == MBO_OK);
        CHECK(fake::held == 0);
    }
}

// A surface whose axis passes or interpolation groups are refused memory is created with
// the cell kernels or the general interpolation.
static void surface_memory()
{
    int cells = 0, general = 0, refused = 0;
    for (int k = 0;; ++k) {
        mbo_surface_t s = nullptr;
        fake::fail_in = k;  // the k-th allocation of the creation, none for 0
        const mbo_status st = mbo_surface_sphere(&s, 1.0, 0.2, 3, 0.01, 1e-4, 2, MBO_F32, nullptr);
        const bool hit = k > 0 && fake::fail_in == 0;
        fake::fail_in = 0;
        CHECK(hit || st == MBO_OK);
        if (!s) {
            CHECK(st == MBO_ERR_ALLOC);
            CHECK(fake::held == 0);
            ++refused;
            continue;
        }
        int64_t m = 0, nc = 0;
        int grid = 0;
        double w = 0.0;
        CHECK(mbo_surface_info(s, &m, &nc, &grid, &w) == MBO_OK);
        std::vector<float> A((size_t)4 * (size_t)m, 1.0f), B(A.size());
        fake::reset();
        CHECK(mbo_surface_diffuse(s, A.data(), B.data()) == MBO_OK);
        const bool sep = fake::count("surface_sep") == 1, gr = fake::count("interp_groups") == 1;
        CHECK(sep || (fake::count("spread_cells") == 1 && fake::count("surface_gather") == 1));
        CHECK(gr || fake::count("surface_interp") == 1);
        CHECK(hit || (sep && gr));
        cells += !sep;
        general += !gr;
        CHECK(mbo_surface_destroy(s) == MBO_OK);
        CHECK(fake::held == 0);
        if (k > 0 && !hit) break;
    }
    CHECK(cells == 1 && general == 1);
    CHECK(refused > 5);
}

// Pinned buffers of small logs outlive their plans: plans that come and go use the same
// one, at most 16 are kept, a large one is the plan's own, and threads share them.
static void pinned_buffers()
{
    const int64_t N[2] = {64, 64};
    std::vector<double> A((size_t)4 * 64 * 64, 1.0), B(A.size());
    auto plan = [&] {
        mbo_plan_t p = nullptr;
        CHECK(mbo_plan(&p, 2, N, 2, 1, 1e-3, MBO_F64, 0.0, nullptr) == MBO_OK);
        return p;
    };
    for (int i = 0; i < 5; ++i) {
        mbo_plan_t p = plan();
        CHECK(mbo_project(p, A.data(), B.data(), nullptr) == MBO_OK);
        CHECK(mbo_plan_destroy(p) == MBO_OK);
    }
    CHECK(fake::host_allocs == 1 && fake::host_frees == 0);
    std::vector<mbo_plan_t> many;
    for (int i = 0; i < 40; ++i) {
        many.push_back(plan());
        CHECK(mbo_project(many.back(), A.data(), B.data(), nullptr) == MBO_OK);
    }
    CHECK(fake::host_allocs == 40);
    for (mbo_plan_t p : many) CHECK(mbo_plan_destroy(p) == MBO_OK);
    CHECK(fake::host_frees == 24);
    mbo_plan_t p = plan();
    std::vector<int64_t> flips(2000);
    CHECK(mbo_iterate(p, A.data(), 2000, 0.0, nullptr, nullptr, flips.data(), nullptr, nullptr) == MBO_OK);
    CHECK(fake::host_allocs == 41);
    CHECK(mbo_plan_destroy(p) == MBO_OK);
    CHECK(fake::host_frees == 25);
    std::vector<std::thread> th;
    for (int t = 0; t < 4; ++t)
        th.emplace_back([&, t] {
            std::vector<double> X((size_t)4 * 64 * 64, 1.0);
            for (int i = 0; i < 20; ++i) {
                mbo_plan_t q = nullptr;
                if (mbo_plan(&q, 2, N, 2, 1, 1e-3, MBO_F64, 0.0, nullptr) != MBO_OK) std::abort();
                double e = 0.0;
                if (mbo_energy(q, X.data(), &e) != MBO_OK) std::abort();
                (void)mbo_plan_destroy(q);
            }
        });
    for (std::thread& t : th) t.join();
    CHECK(fake::host_allocs == 41 && fake::host_frees == 25);
    CHECK(fake::held == 0);
}

// The device word of the field's pointer is written on the stream that reads it: also
// when a call that wrote it ended early on another stream.
static void field_word()
{
    const int64_t N[2] = {64, 64};
    std::vector<double> A((size_t)2 * 4 * 64 * 64, 1.0);
    hipStream_t s1 = nullptr, s2 = nullptr;
    CHECK(hipStreamCreateWithFlags(&s1, 0) == hipSuccess && hipStreamCreateWithFlags(&s2, 0) == hipSuccess);
    auto at = [](const char* n, hipStream_t s) { return std::string(n) + "@" + std::to_string((unsigned long long)(uintptr_t)s); };
    for (int batched = 0; batched < 2; ++batched) {
        mbo_plan_t p = nullptr;
        if (batched) {
            mbo_field_desc d[2];
            std::memset(d, 0, sizeof d);
            for (int i = 0; i < 2; ++i) {
                d[i].d = 2;
                d[i].N[0] = d[i].N[1] = 64;
                d[i].n = 2;
                d[i].tau = 1e-3;
            }
            CHECK(mbo_plan_batched(&p, 2, d, MBO_F64, 0.0, 0, s1) == MBO_OK);
        } else {
            CHECK(mbo_plan(&p, 2, N, 2, 1, 1e-3, MBO_F64, 0.0, s1) == MBO_OK);
        }
        if (!p) return;
        fake::fail_instantiate = true;
        CHECK(mbo_iterate(p, A.data(), 2, 0.0, nullptr, nullptr, nullptr, nullptr, nullptr) != MBO_OK);
        fake::fail_instantiate = false;
        fake::reset();
        CHECK(mbo_plan_set_stream(p, s2) == MBO_OK);
        CHECK(mbo_iterate(p, A.data(), 2, 0.0, nullptr, nullptr, nullptr, nullptr, nullptr) == MBO_OK);
        CHECK(fake::count("set_slot") == 1 && fake::order.front() == at("set_slot", s2));
        CHECK(mbo_iterate(p, A.data(), 2, 0.0, nullptr, nullptr, nullptr, nullptr, nullptr) == MBO_OK);
        CHECK(fake::count("set_slot") == 1);
        CHECK(mbo_plan_destroy(p) == MBO_OK);
    }
    CHECK(hipStreamDestroy(s1) == hipSuccess && hipStreamDestroy(s2) == hipSuccess);
    CHECK(fake::held == 0);
}

int main(int argc, char** argv)
{
    const char* s = argc > 1 ? argv[1] : "";
    if (!std::strcmp(s, "set_tau_2d")) set_tau(2);
    else if (!std::strcmp(s, "set_tau_3d")) set_tau(3);
    else if (!std::strcmp(s, "volume_memory")) volume_memory();
    else if (!std::strcmp(s, "adjoint_memory")) adjoint_memory();
    else if (!std::strcmp(s, "surface_memory")) surface_memory();
    else if (!std::strcmp(s, "pinned_buffers")) pinned_buffers();
    else if (!std::strcmp(s, "field_word")) field_word();
    else return 2;
    if (!bad) std::printf("ok\n");
    return bad;
}

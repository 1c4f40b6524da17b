// Host side of plans under refused allocations and changed streams (fake_runtime.hpp).
// Each scenario prints "ok" or what went wrong; run by tests/test_host_runtime.py.
#include <cmath>
#include <cstdio>
#include <cstring>
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

int main(int argc, char** argv)
{
    const char* s = argc > 1 ? argv[1] : "";
    if (!std::strcmp(s, "set_tau_2d")) set_tau(2);
    else if (!std::strcmp(s, "set_tau_3d")) set_tau(3);
    else return 2;
    if (!bad) std::printf("ok\n");
    return bad;
}

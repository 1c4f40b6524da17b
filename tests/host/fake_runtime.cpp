#include "fake_runtime.hpp"

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>

namespace fake {
int fail_in = 0;
bool fail_instantiate = false;
size_t fail_above = 0, held = 0;
std::map<std::string, int> launches;
std::vector<std::string> order;
mbo::FastColArgs heat;
int host_allocs = 0, host_frees = 0;
static std::map<void*, size_t> size_of;
static std::mutex mutex;
static hipError_t last = hipSuccess;  // until hipGetLastError, also by the next launcher

static hipError_t note(const char* name, hipStream_t st, bool prepare = false)
{
    if (prepare) return hipSuccess;
    std::lock_guard<std::mutex> lock(mutex);
    ++launches[name];
    order.push_back(std::string(name) + "@" + std::to_string((unsigned long long)(uintptr_t)st));
    return hipGetLastError();
}
}  // namespace fake

extern "C" {
hipError_t hipMalloc(void** p, size_t n)
{
    std::lock_guard<std::mutex> lock(fake::mutex);
    if (fake::fail_in > 0 && --fake::fail_in == 0) return fake::last = hipErrorOutOfMemory;
    if (fake::fail_above && n > fake::fail_above) return fake::last = hipErrorOutOfMemory;
    *p = std::malloc(n ? n : 1);
    fake::size_of[*p] = n;
    fake::held += n;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    std::lock_guard<std::mutex> lock(fake::mutex);
    if (p) {
        fake::held -= fake::size_of.at(p);
        fake::size_of.erase(p);
        std::free(p);
    }
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    std::lock_guard<std::mutex> lock(fake::mutex);
    ++fake::host_allocs;
    *p = std::calloc(n ? n : 1, 1);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    std::lock_guard<std::mutex> lock(fake::mutex);
    ++fake::host_frees;
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n)
{
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    std::memset(p, 0, sizeof *p);
    p->sharedMemPerBlock = 160 * 1024;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetLastError()
{
    const hipError_t e = fake::last;
    fake::last = hipSuccess;
    return e;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = (hipStream_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    std::free(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    *g = (hipGraph_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t)
{
    if (fake::fail_instantiate) return fake::last = hipErrorOutOfMemory;
    *e = (hipGraphExec_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t st) { return fake::note("graph", st); }
hipError_t hipGraphDestroy(hipGraph_t g)
{
    std::free(g);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e)
{
    std::free(e);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    std::free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t)
{
    *ms = 1.0f;
    return hipSuccess;
}
}  // extern "C"

namespace mbo {
using fake::note;

hipError_t launch_row(int, int, int, const RowArgs&, dim3, dim3, size_t, hipStream_t st, bool prepare, hipEvent_t,
                      hipEvent_t)
{
    return note("row", st, prepare);
}
hipError_t launch_col(int, int, int, const ColArgs&, dim3, dim3, size_t, hipStream_t st, bool prepare, hipEvent_t,
                      hipEvent_t)
{
    return note("col", st, prepare);
}
hipError_t launch_project(int, int, const ProjArgs&, int, hipStream_t st) { return note("project", st); }
hipError_t launch_fill_u64(unsigned long long* p, int64_t n, unsigned long long v, hipStream_t st)
{
    for (int64_t i = 0; i < n; ++i) p[i] = v;
    return note("fill", st);
}
hipError_t launch_fill_i32(int* p, int64_t n, int v, hipStream_t st)
{
    for (int64_t i = 0; i < n; ++i) p[i] = v;
    return note("fill", st);
}
hipError_t launch_reduce(const ReduceArgs&, hipStream_t st) { return note("reduce", st); }
hipError_t launch_init_logs(unsigned long long* p, int64_t n, int* stop, int batch, int K, hipStream_t st)
{
    for (int64_t i = 0; i < n; ++i) p[i] = 0;
    for (int i = 0; i < batch; ++i) stop[i] = K;
    return note("init_logs", st);
}
hipError_t launch_export(unsigned long long* d, unsigned long long* s, int64_t n, const unsigned long long*, int64_t,
                         bool, hipStream_t st)
{
    std::memcpy(d, s, (size_t)n * 8);
    return note("export", st);
}
hipError_t launch_set_slot(void** slot, void* p, hipStream_t st)
{
    *slot = p;
    return note("set_slot", st);
}
hipError_t launch_vjp(int, int, const VjpArgs&, int, hipStream_t st) { return note("vjp", st); }
hipError_t launch_fill_uniform(int, void*, int64_t, uint64_t, hipStream_t st) { return note("uniform", st); }
hipError_t launch_so2_index(int, const void*, int64_t, int64_t, int, int, double*, hipStream_t st)
{
    return note("so2", st);
}
hipError_t launch_sum_rows(const double*, int64_t, int, double*, hipStream_t st, bool) { return note("sum_rows", st); }
hipError_t launch_select(int, const SelArgs&, int, hipStream_t st) { return note("select", st); }
hipError_t launch_select_list(int, const SelListArgs&, int, hipStream_t st) { return note("select_list", st); }
hipError_t launch_sel_mark(int, const SelArgs&, int, hipStream_t st) { return note("sel_mark", st); }
hipError_t launch_count_pos(const int8_t*, int64_t, int, long long*, hipStream_t st) { return note("count_pos", st); }
hipError_t launch_row_vp(int, int, int, const RowArgs&, dim3, dim3, size_t, hipStream_t st, bool prepare)
{
    return note("row_vp", st, prepare);
}
hipError_t launch_surface_sep(int, const SurfSepArgs&, hipStream_t st, size_t prepare_lds)
{
    return note("surface_sep", st, prepare_lds != 0);
}
int sep_tile(int len_x, int len_y, size_t esz, size_t lds_max)
{
    return (size_t)2 * ((len_x > len_y ? len_x : len_y) + 16) * esz * 8 <= lds_max ? 8 : 0;
}
size_t sep_z_lds(int, int, int, size_t) { return 0; }
hipError_t launch_surface_interp_groups(int, const SurfArgs&, const SurfGroup*, int, hipStream_t st)
{
    return note("interp_groups", st);
}
hipError_t launch_surface_spread(int, const SurfArgs&, hipStream_t st) { return note("surface_spread", st); }
hipError_t launch_surface_spread_cells(int, const SurfArgs&, int, hipStream_t st) { return note("spread_cells", st); }
hipError_t launch_surface_interp(int, const SurfArgs&, hipStream_t st) { return note("surface_interp", st); }
hipError_t launch_surface_gather(int, const SurfArgs&, int, hipStream_t st) { return note("surface_gather", st); }
hipError_t launch_surf_vp_key(int, int, const SurfVolArgs&, hipStream_t st) { return note("surf_vp_key", st); }
hipError_t launch_wsel(int, const SurfVolArgs&, long long, long long, hipStream_t st) { return note("wsel", st); }
hipError_t launch_wsel_mark(int, const SurfVolArgs&, hipStream_t st) { return note("wsel_mark", st); }
hipError_t launch_surf_vp_apply(int, int, const SurfVolArgs&, hipStream_t st) { return note("surf_vp_apply", st); }
hipError_t launch_row_relax(int, int, int, const RowArgs&, dim3, dim3, size_t, hipStream_t st, bool prepare)
{
    return note("row_relax", st, prepare);
}
hipError_t launch_penalty(int, int, const void*, int64_t, int, int, double*, hipStream_t st) { return note("penalty", st); }
hipError_t launch_row_fast(int, int, int, const FastRowArgs&, dim3, hipStream_t st, bool prepare, hipEvent_t, hipEvent_t)
{
    return note("row_fast", st, prepare);
}
hipError_t launch_heat_fast(int, int, int, const FastColArgs& a, dim3, hipStream_t st, bool prepare, hipEvent_t,
                            hipEvent_t)
{
    if (!prepare) fake::heat = a;
    return note("heat_fast", st, prepare);
}
bool row_fast_vjp_served(int prec, int n) { return n == 2 || (n == 3 && prec == 1); }
hipError_t launch_row_fast_vjp(int, int, int, const FastRowArgs&, dim3, hipStream_t st, bool prepare)
{
    return note("row_fast_vjp", st, prepare);
}
hipError_t launch_heat_fast_adj(int, int, int, const FastColArgs&, dim3, hipStream_t st, bool prepare)
{
    return note("heat_fast_adj", st, prepare);
}
int heat_fast_adj_tile(int log2L) { return log2L >= 8 ? 2 : 512 >> log2L; }
hipError_t launch_row_fast_vkey(int, int, int, const FastRowArgs&, dim3, hipStream_t st, bool prepare)
{
    return note("row_fast_vkey", st, prepare);
}
hipError_t launch_volume_fix(int, int, const VolFixArgs&, dim3, hipStream_t st) { return note("volume_fix", st); }
hipError_t launch_volume_redo(int, int, int, const VolFixArgs&, dim3, hipStream_t st, bool prepare)
{
    return note("volume_redo", st, prepare);
}
hipError_t launch_row_fast_relax(int, int, int, const FastRowArgs&, dim3, hipStream_t st, bool prepare)
{
    return note("row_fast_relax", st, prepare);
}
hipError_t launch_resolvent_fast(int, int, const FastColArgs&, dim3, hipStream_t st, bool prepare)
{
    return note("resolvent_fast", st, prepare);
}
int resolvent_fast_tile(int log2L) { return log2L >= 11 ? 2 : log2L >= 8 ? 4 : 512 >> log2L; }
hipError_t launch_plane_fast(int, int, int, const FastColArgs& a, dim3, hipStream_t st, bool prepare, hipEvent_t,
                             hipEvent_t)
{
    if (!prepare) fake::heat = a;
    return note("plane_fast", st, prepare);
}
int plane_fast_group(int log2Y, int log2Z)
{
    const int t = (1 << (log2Y + log2Z)) / 16;
    return t < 64 ? 64 / t : 1;
}
int plane_fast_threads(int log2Y, int log2Z) { return plane_fast_group(log2Y, log2Z) * ((1 << (log2Y + log2Z)) / 16); }
size_t plane_fast_lds_bytes(int prec, int log2Y, int log2Z)
{
    return ((size_t)plane_fast_group(log2Y, log2Z) << log2Z) * ((1 << log2Y) + 1) * (prec == 1 ? 8 : 16);
}
hipError_t launch_sum_counts(const unsigned long long*, int, int, int, int, unsigned long long*, unsigned long long*,
                             unsigned long long*, hipStream_t st)
{
    return note("sum_counts", st);
}
size_t row_fast_lds_bytes(int prec, int n, int log2L)
{
    const int L = 1 << log2L, rows = L >= 512 ? 1 : 512 / L;
    return (size_t)rows * ((n * n + 1) / 2) * (L + L / 8) * (prec == 1 ? 8 : 16);
}
int row_fast_rows_per_group(int log2L) { return log2L >= 9 ? 1 : 512 >> log2L; }
}  // namespace mbo

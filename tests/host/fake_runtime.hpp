// A HIP runtime and kernel launchers on host memory, for tests of the host side of the
// C ABI (mbo_api.cpp) without a GPU: allocations are malloc, copies memcpy, launches
// only recorded.  A test says which allocations fail.
#pragma once
#include <cstddef>
#include <map>
#include <string>
#include <vector>

#include "mbo_internal.hpp"

namespace fake {
extern int fail_in;               // > 0: the fail_in-th hipMalloc from now is refused
extern size_t fail_above;         // > 0: every hipMalloc of more bytes is refused
extern bool fail_instantiate;     // hipGraphInstantiate is refused
extern std::map<std::string, int> launches;  // by launcher
extern std::vector<std::string> order;       // the launches in order, with their stream ("name@stream")
extern mbo::FastColArgs heat;     // arguments of the last launch_heat_fast
extern size_t held;               // bytes of device memory in use
extern int host_allocs, host_frees;  // of pinned memory
inline int count(const std::string& n) { return launches.count(n) ? launches[n] : 0; }
inline void reset()
{
    launches.clear();
    order.clear();
}
}  // namespace fake

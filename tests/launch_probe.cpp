// The library's planner and launch code (kvx_plan.cpp) with the HIP runtime
// and the kernels replaced: device memory is host memory, and a launch keeps
// its arguments instead of running.  tests/test_launch_forms.py builds it with
// g++ into a shared library, makes the public launch calls on a CPU and reads
// which kernel form and which stores the planner's rules chose, and which rows
// the launch's workgroups would take.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>

#include "kvx.h"
#include "kvx_host.h"
#include "kvx_internal.h"

namespace {
kvx::KArgs g_args;
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n)
{
    *p = std::malloc(n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
}

namespace kvx {
int launch(int, int, int, const KArgs& a, void*) { g_args = a; return 0; }
int scratch_items(Item**) { return int(hipErrorNoDevice); }
int build_items(const ItemsArgs&, void*) { return int(hipErrorNoDevice); }
}  // namespace kvx

extern "C" {

// The last launch: form, store, work units, and what the
// walk's index space is (planes, pages per plane, segments, rows of a page in
// its widest segment, chunks per row).
int probe_launch(int64_t* out)
{
    const kvx::Args& a = g_args.a;
    int n = a.seg0.n;
    for (uint32_t j = 1; j < a.num_segs; ++j) n = g_args.seg[j].n > n ? g_args.seg[j].n : n;
    const int64_t v[] = {g_args.form, a.store, a.units, a.planes, a.num_items,
                         a.num_segs, int64_t(a.block_size) * n, a.cpr};
    std::memcpy(out, v, sizeof v);
    return int(sizeof v / sizeof v[0]);
}

}

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

// Counts in hits[plane][page][segment][row][chunk] how often the last launch's
// lanes take each 16-byte chunk of a row that exists.  The lanes of a unit are
// those of the kernels (units dealt to the XCDs in runs; page-aligned or flat).
// Returns 0, or what is wrong: 1 an index outside its range, 2 more units than
// a launch may have, 3 a page of the only request that is not the plan's item,
// 4 a quantising row that is not held by aligned lanes.
int probe_walk(const kvx_plan_t* p, const int32_t* bt, int32_t bt_stride, int aligned_rows,
               uint8_t* hits)
{
    const kvx::KArgs& k = g_args;
    const kvx::Args& a = k.a;
    auto div = [](uint32_t n, kvx::FastDiv f) {
        return uint32_t(((uint64_t(n) * f.mul >> 32) + n) >> f.shift);
    };
    int max_n = a.seg0.n;
    for (uint32_t j = 1; j < a.num_segs; ++j) max_n = k.seg[j].n > max_n ? k.seg[j].n : max_n;
    const int64_t page_rows = int64_t(a.block_size) * max_n;
    const uint32_t grid = a.units_per_xcd * kvx::kXcds;
    if (int64_t(grid) > kvx::kMaxUnits + kvx::kXcds) return 2;
    for (uint32_t block = 0; block < grid; ++block) {
        const uint32_t unit = (block % kvx::kXcds) * a.units_per_xcd + block / kvx::kXcds;
        if (unit >= a.units) continue;
        for (uint32_t tid = 0; tid < uint32_t(kvx::kThreads); ++tid) {
            uint32_t plane, sg, item, part = 0;
            int64_t sub, r;
            if (k.form != kvx::kAligned) {
                const uint32_t q1 = div(unit, a.div_segs);
                sg = unit - q1 * a.num_segs;
                plane = div(q1, a.div_parts);
                const uint32_t slot = (q1 - plane * a.parts) * kvx::kThreads + tid;
                const uint32_t row = div(slot, k.b.div_row_lanes);
                sub = slot - row * k.b.row_lanes;
                item = div(row, k.b.div_page_rows);
                r = row - item * k.b.page_rows;
                if (aligned_rows && (tid - sub) % k.b.row_lanes) return 4;
                if (item >= a.num_items) continue;
            } else {
                const uint32_t q1 = div(unit, a.div_parts);
                part = unit - q1 * a.parts;
                const uint32_t q2 = div(q1, a.div_segs);
                sg = q1 - q2 * a.num_segs;
                plane = div(q2, a.div_items);
                item = q2 - plane * a.num_items;
                if (item >= a.num_items) return 1;
                sub = tid & ((1u << a.lg_lpr) - 1);
                r = int64_t(part) * (kvx::kThreads >> a.lg_lpr) + (tid >> a.lg_lpr);
            }
            if (plane >= a.planes || sg >= a.num_segs) return 1;
            kvx::Item it;
            const kvx::Item& want = p->items[item];
            const int32_t* row_of_table = a.bt;
            if (a.one_tokens) {
                it = kvx::Item{0, 0, a.one_wire_scale, 0, int32_t(item), a.one_tokens, 0};
            } else {
                it = a.items[item];
                if (row_of_table) row_of_table += int64_t(it.req) * a.bt_stride;
            }
            if (it.src_base != want.src_base || it.wire_data != want.wire_data ||
                it.wire_scale != want.wire_scale || it.blk != want.blk || it.tokens != want.tokens)
                return 3;
            if (row_of_table && row_of_table != bt + int64_t(want.req) * bt_stride) return 3;
            const kvx::Segment& seg = a.num_segs > 1 ? k.seg[sg] : a.seg0;
            const int64_t t0 = int64_t(it.blk) * a.block_size;
            const int64_t left = it.tokens - t0;
            const int64_t rows = (left < a.block_size ? left : a.block_size) * seg.n;
            if (sub >= a.cpr || r >= rows) continue;
            if (r >= page_rows) return 1;
            ++hits[(((int64_t(plane) * a.num_items + item) * a.num_segs + sg) * page_rows + r) * a.cpr + sub];
        }
    }
    return 0;
}

}

// Internal declarations shared by the host planner (kvx_plan.cpp) and the
// gfx950 kernels (kvx_kernels.hip).
#pragma once

#include <cstdint>

#include "kvx.h"

namespace kvx {

constexpr int kThreads = 256;           // threads per workgroup (4 wave64)
constexpr int kMaxHeadsPerRank = 1024;  // Hd limit
constexpr int kMaxReadShards = 64;      // head segments (and so source shards) of a decode rank
constexpr int kMaxRowChunks = 64;       // 16-byte destination chunks per row (one wave)
constexpr int kXcds = 8;                // MI355X: workgroups are dealt round-robin to 8 XCDs
// work units of one launch; the 1-D grid is this rounded up to a multiple of
// kXcds, and grid * kThreads stays below 2^32
constexpr int64_t kMaxUnits = (int64_t(1) << 24) - kXcds;

// Division by an invariant divisor d >= 1 (Granlund and Montgomery, 1994):
// n / d = (mulhi(n, mul) + n) >> shift for every 32-bit n, with
// shift = ceil(log2 d) and mul = floor(2^32 (2^shift - d) / d) + 1.
struct FastDiv {
    uint32_t mul;
    uint32_t shift;
};

// One logical page of one request, device resident: the unit of work of a
// workgroup in every (layer, k/v) plane.
struct Item {
    int64_t src_base;    // element offset of the request in every source shard (0 if paged)
    int64_t wire_data;   // byte offset of the request's data region in the transfer tensor
    int64_t wire_scale;  // byte offset of its scale region, -1 without scales
    int32_t req;         // request index (block-table row)
    int32_t blk;         // page index within the request
    int32_t tokens;      // T_r
    int32_t pad;
};

enum Mode : int { kPack = 0, kUnpack = 1, kRepack = 2 };

// element conversion performed by a launch
enum Conv : int {
    kCopy16 = 0,    // 16-bit bits unchanged
    kF16Bf16 = 1,   // fp16 -> bf16, round to nearest even
    kBf16E4m3 = 2,  // bf16 -> e4m3fn with per-row scale
    kF16E4m3 = 3,   // fp16 -> e4m3fn with per-row scale
    kCopy8 = 4,     // 8-bit bits unchanged (+ scale copy), unpack of an 8-bit format
    kBf16F16 = 5,   // bf16 -> fp16, round to nearest even, overflow to infinity
    // dequantising unpack: e4m3fn transfer tensor (+ scales) -> 16-bit cache
    kDq8Bf16 = 6,
    kDq8F16 = 7,
    // repack into a 16-bit cache through e4m3fn: quantise, then dequantise
    kQdBf16Bf16 = 8,
    kQdF16Bf16 = 9,
    kQdBf16F16 = 10,
    kQdF16F16 = 11,
    // the same with OCP e5m2 codes (scale max|x| / 57344)
    kBf16E5m2 = 12,
    kF16E5m2 = 13,
    kDq5Bf16 = 14,
    kDq5F16 = 15,
    kQd5Bf16Bf16 = 16,
    kQd5F16Bf16 = 17,
    kQd5Bf16F16 = 18,
    kQd5F16F16 = 19
};

// A run of the decode rank's heads that comes from one source shard: decode
// heads [i0, i0 + n) are heads [h0, h0 + n) of that shard.
struct Segment {
    const void* src;                  // the shard (launches; the unpack's transfer tensor)
    int32_t slot;                     // the shard's place among the shards that are read
    int32_t h0;
    int32_t i0;
    int32_t n;
    FastDiv div_n;
};

// Cache policy of the destination rows' stores.
enum Store : int { kStoreStream = 0, kStoreThrough = 1, kStoreCached = 2 };

// Units of page-aligned workgroups, or the rows of consecutive pages packed
// into workgroups, written with kStoreStream or kStoreCached.
enum Form : int { kAligned = 0, kFlat = 1, kFlatCached = 2 };

// Kernel arguments (passed by value through the kernel-argument segment).  The
// page-aligned form reads the groups that it needs whole, at its start, so that
// one wait covers them all: Args and, for paged sources, ArgsPaged; a launch
// with one head segment does not read seg[].
struct Args {
    uint32_t units;                   // work units: planes x pages x segments x parts
    uint32_t units_per_xcd;           // grid / kXcds
    uint32_t num_segs;
    uint32_t num_items;               // logical pages per plane
    uint32_t planes;                  // 2 x converted layers
    uint32_t parts;                   // workgroup passes per (page, segment); flat launches:
                                      // workgroups per plane and segment
    FastDiv div_parts, div_segs, div_items;
    const Item* items;
    const int32_t* bt;
    int32_t bt_stride;
    int32_t block_size;
    int32_t hs;                       // heads per source shard
    int32_t hd;                       // heads per decode rank
    int32_t head_dim;
    int32_t cpr;                      // 16-byte transfer-tensor chunks per row
    int16_t lg_lpr;                   // log2(lanes per row), lanes per row >= cpr
    int16_t store;                    // Store: how destination rows are written (kAligned)
    int32_t row_dst_bytes;            // pack: transfer-tensor row bytes; else cache row bytes
    uint32_t src_plane0;              // 2 x source layer offset (pipeline stages)
    uint32_t dst_plane0;              // 2 x cache layer offset
    void* dst;                        // pack: transfer tensor; else cache
    int64_t num_blocks;
    int64_t plane_bytes;              // cache bytes per (layer, k/v) plane
    Segment seg0;                     // the only head segment where num_segs is 1
    int32_t one_tokens;               // tokens of the only request with pages, 0: items[] holds them
    int32_t row_wire_bytes;           // transfer-tensor row bytes (the unpack's source rows)
    int64_t one_wire_scale;           // that request's Item::wire_scale (its other offsets are 0)
    float* dscale;                    // cache scales (unpack/repack into an 8-bit cache)
    int64_t plane_scales;             // cache scales per plane
};

struct ArgsFlat {                     // flat launches: the rows of a plane's pages
                                      // packed into workgroups
    uint32_t row_lanes;               // lanes per row: cpr, or the power of two above it
    uint32_t page_rows;               // rows of a page in its widest segment
    FastDiv div_row_lanes, div_page_rows;
};

struct ArgsPaged {                    // paged sources: the prefill side's pages
    const int32_t* sbt;               // source block table [requests][sbt_stride]
    int64_t src_num_blocks;           // pages per plane of each shard's pool
    int32_t sbt_stride;
    int32_t src_block_size;
    FastDiv div_sbs;
    int32_t sbt_uniform;              // every part lies in one source page
    int32_t pad;
};

struct KArgs {
    Args a;
    ArgsFlat b;
    ArgsPaged p;
    int32_t form;                     // Form: which kernel (read by the host)
    int32_t pad;
    Segment seg[kMaxReadShards];      // the head segments, where there is more than one
};
static_assert(sizeof(Args) == 192 && sizeof(ArgsFlat) == 24 && sizeof(ArgsPaged) == 40,
              "the kernels read the argument groups as whole dwords");

// Launch one conversion over the arguments' work units; returns a hipError_t value.
int launch(int mode, int conv, int order, const KArgs& a, void* stream);

// The allocation-free repack keeps its work-item table in a static device
// array of kNoAllocItems entries (40 B each: 2.5 MiB per device) and takes at
// most kNoAllocRequests requests, whose lengths travel in the arguments of the
// kernel that writes that table.
constexpr int kNoAllocItems = 65536;
constexpr int kNoAllocRequests = 256;

struct ItemsArgs {
    int32_t lens[kNoAllocRequests];   // tokens per request
    int32_t num_requests;
    int32_t block_size;               // destination page size
    int32_t num_items;                // items of the table
    int32_t pad;
    int64_t src_elems_per_token;      // elements of one token in a source shard (2 x layers x Hs x D)
    Item* items;                      // the table to write
};

// The current device's static work-item table; the address is looked up once
// per device.  Returns a hipError_t value.
int scratch_items(Item** out);

// Enqueue the kernel that writes the work-item table of a.lens (one page of
// a request per item, requests in order) on `stream`.  Returns a hipError_t
// value.
int build_items(const ItemsArgs& a, void* stream);

FastDiv make_fastdiv(uint32_t d);

}  // namespace kvx

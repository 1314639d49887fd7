// The tile copy behind llmig_stage, llmig_pack and llmig_unpack, with its
// launch configuration.  Part of the single translation unit built from
// llmig.hip.
//
// What it computes (Llumnix §4.2, §5 "Block fusion"): for every pair i, layer
// l and K/V, the tile_bytes of tile (l, kv) of block src[i] land in tile
// (l, kv) of block dst[i] (pool to pool), or in slot ((l * 2 + kv) * n + i)
// of a contiguous staging buffer (pack), or the reverse (unpack).
//
// Two kernels, chosen by whether the caller caps the grid:
//
// copy_rows, every uncapped launch.  A call's bytes are a list of 1 KiB rows
// (64 lanes x 16 bytes); a wavefront moves one row, one load and one store per
// lane, and is a workgroup by itself (a small launch: two rows, two wavefronts).
//  * What bounds it is HBM, and how well DRAM likes the order in which a
//    launch touches it.  With one row per wavefront the rows in flight at any
//    time (32 wavefronts a CU, 8 MiB over the chip) are consecutive in the
//    launch's order, so they fall into few DRAM pages; with more rows per
//    wavefront each wavefront walks a run of its own and the same bytes in
//    flight are spread over thousands of runs.  Measured on MI355X, one
//    process, read + written bytes, 4 / 32 / 52 / 128 KiB tiles: 1 row 6.5 /
//    6.7 / 6.7 / 6.85 TB/s, 2 rows 6.1 / 5.8 / 6.2 / 6.2, 4 rows 5.6 / 5.5 /
//    5.7 / 5.8; spans of a quarter tile walked pair by pair (copy_tiles, what
//    ran before) 5.0 / 5.1 / 5.7 / 6.25.
//  * The order is plane-major: all pairs of one (layer, K/V) tensor, then
//    the next tensor.  Pair-major order spreads neighbouring rows over 2 *
//    num_layers tensors (4 KiB tiles: 5.0 against 5.9-6.3 TB/s).
//  * The pairs of a bulk call with ids on the host are ordered by destination
//    block (order_pairs), so that the writes of a tensor sweep it upwards:
//    +2-9% over random pairs on tiles up to 64 KiB, +1% on 128 KiB (ordering
//    by source instead gains half of that or less; ordering launch by launch
//    of 512 pairs loses half of it from 2000 pairs on).  The order is free: no
//    destination block occurs twice in a call.
//  * Consecutive rows go to the eight XCDs in turn, the dispatcher's own
//    order, for tiles below 128 KiB; from there on each XCD takes runs of
//    kXcdRun rows (128 KiB tiles 6.63 -> 6.84, 256 KiB 6.75 -> 6.81, but
//    64 KiB 6.69 -> 6.66 and 32 KiB 6.66 -> 6.44 TB/s).
//  * A launch of at most one round of resident wavefronts (a final stage of
//    a block or so) moves two rows per wavefront: it has no DRAM order to
//    keep, and half as many wavefronts to dispatch (one block of 60 layers of
//    52 KiB tiles 4.87 against 5.10 us, of 80 layers of 32 KiB 4.27 against
//    4.63 us, of 32 layers of 128 KiB 5.03 against 5.09 us; 4000 pairs of 2 KiB
//    tiles of 2 layers through a staging buffer in HBM, 32 launches, 106
//    against 110 us).  Its workgroups are two wavefronts, half as many again to
//    dispatch: whole finishing passes, each with a write and a stage of one
//    block of 128 KiB tiles, 19 layers 23.4 -> 22.6 us, 24 layers 24.0 -> 23.2,
//    28 layers 24.2 -> 23.5; other tiles and staging in HBM level (four
//    wavefronts: the same).  With the staging buffer in host memory it keeps one:
//    two were 1-3% slower over the link (six pieces of 2.6 MB of 128 KiB tiles
//    each way 723 against 702 us, one of 3.9 MB of 16 KiB tiles 216 against
//    210 us).
//
// copy_tiles, launches under a workgroup cap (the throttle of a migration's
// non-final stages).  Few resident workgroups walk the items, so each must
// keep many bytes in flight by itself:
//  * A tile is cut into SPAN-KiB spans and each span is one wavefront's work
//    item: the wave issues SPAN 1-KiB loads before its first store.  SPAN is
//    about a quarter of the tile, so the four wavefronts of a workgroup move
//    one whole tile.  Items run pair-major.
//  * Every span runs the same unpredicated sequence of SPAN loads and SPAN
//    stores.  A row of the span that lies past the end of the tile (the
//    last span of a tile that is not a whole number of spans, such as the
//    4 KiB tail of a 52 KiB tile cut into 16 KiB spans) gets an offset past
//    the buffer resource's range, so the hardware's range check returns
//    zeros for its load and drops its store.  Predicating those rows on
//    the lane mask instead makes the compiler wait for every earlier memory
//    operation before each store of the span (it cannot count them across
//    the branches), which serialised the tail's stores.
//
// Both:
//  * The block ids of an item are wavefront-uniform; they and the per-layer
//    base addresses are read with scalar loads, so the only vector memory
//    traffic is the copy itself.
//  * A stage's (src, dst) ids travel inside the kernel arguments, so a
//    stage needs no mapping upload and no device allocation: the short
//    final stage costs one launch.  When every id of a pool-to-pool stage
//    fits in 16 bits (pools of up to 65536 blocks) a pair takes one 32-bit
//    word and a launch carries 2 * kInlinePairs pairs (the whole 512-pair
//    LLaMA-7B stage in one launch, measured 0.4-0.7% faster than two);
//    otherwise kInlinePairs pairs of 32-bit ids.
//  * No LDS: both sides have the same byte layout inside a tile, so data
//    goes straight from the load registers to the store.  No MFMA: a copy
//    has no arithmetic.
//  * Loads and stores are raw buffer accesses over one tile with explicit
//    cache policy: non-temporal loads, and stores that are non-temporal
//    with the sc1 scope bit (device scope on gfx950).  Every byte is touched
//    once, and streaming it past the caches leaves them to the decode work
//    beside the migration.  (copy_rows, 32 KiB tiles: 6.43 TB/s; cached
//    loads 6.12, plain stores 5.5, sc1 stores without nt 5.7.)
#pragma once

#include <algorithm>
#include <vector>

#include "common.h"

namespace {

enum Side { kPool = 0, kLinear = 1 };


// Arguments of one copy launch.  Pool sides address tile (l, kv, id) at
// tab[kv * L + l] + id * tile_bytes; linear sides address tile x of plane
// (l, kv) at lin + ((l * 2 + kv) * lin_pairs + x) * tile_bytes.  For pair i
// of the launch, x is lin_first + i, or, for a linear source whose pairs
// were reordered, the pair's place in the call, which then rides as its source
// id (kIds32).
struct CopyArgs {
    const uint64_t *src_tab;
    const uint64_t *dst_tab;
    const uint8_t *src_lin;
    uint8_t *dst_lin;
    const int32_t *src_ids_dev; // device id lists (null when the ids are inline)
    const int32_t *dst_ids_dev;
    uint32_t tile_bytes;
    uint32_t num_layers;
    uint32_t planes;            // 2 * num_layers
    uint32_t pairs;             // pairs in this launch
    uint32_t spans_per_tile;
    uint32_t items;             // wave items: pairs * planes * spans_per_tile
    uint32_t first_item;        // this launch's first item (copy_rows)
    Divisor by_span, by_pair;   // division by spans_per_tile and by pairs (copy_rows)
    uint32_t xcd_runs;          // copy_rows: 1 if each XCD takes runs of kXcdRun items
    uint32_t lin_first;         // this launch's first pair within the whole call
    uint32_t lin_pairs;         // pairs in the whole call
    uint32_t ids[2 * kInlinePairs]; // inline ids, laid out as the launch's Ids mode says
};

constexpr uint32_t kWaveRow = 64 * 16;         // one wavefront load: 1 KiB

// Buffer offset of the row starting at byte o of a tile of `bytes` bytes:
// o itself, or kOutOfRange when the row lies past the tile.  A row that is partly inside the tile (a tile that is not a whole number
// of KiB) is cut per lane by the same check.
__device__ __forceinline__ uint32_t row_offset(uint32_t o, uint32_t bytes)
{
    return o < bytes ? o : kOutOfRange;
}

template <int IDS>
__device__ __forceinline__ uint32_t src_id(const CopyArgs &a, uint32_t i)
{
    if (IDS == kIds16)
        return a.ids[i] & 0xffffu;
    return IDS == kIds32 ? a.ids[i] : static_cast<uint32_t>(id_entry(a.src_ids_dev, i));
}

template <int IDS>
__device__ __forceinline__ uint32_t dst_id(const CopyArgs &a, uint32_t i)
{
    if (IDS == kIds16)
        return a.ids[i] >> 16;
    return IDS == kIds32 ? a.ids[kInlinePairs + i] : static_cast<uint32_t>(id_entry(a.dst_ids_dev, i));
}

// Workgroups (rows) in a row on one XCD under xcd_runs: 512 KiB.
constexpr uint32_t kXcdRun = 512;

// ROWS wavefronts per workgroup, one item of ROWS KiB of a tile each.  (A launch's
// items are a multiple of its planes, K and V of each layer, so two wavefronts
// leave none over.  Two rows: a small launch, of less than a round of XCD runs.)
template <int SRC, int DST, int IDS, int ROWS>
__global__ void __launch_bounds__(64 * ROWS) copy_rows(const CopyArgs a)
{
    uint32_t w = ROWS == 1 ? blockIdx.x : uniform(blockIdx.x * ROWS + threadIdx.x / 64);
    if (ROWS == 1 && a.xcd_runs) {
        // the dispatcher hands workgroup g to XCD g % 8: renumbered so that
        // the k-th kXcdRun workgroups of an XCD are consecutive items (the
        // grid's tail keeps the plain order)
        const uint32_t round = w / (8u * kXcdRun), r = w % (8u * kXcdRun);
        if ((round + 1u) * (8u * kXcdRun) <= gridDim.x)
            w = round * (8u * kXcdRun) + (r % 8u) * kXcdRun + r / 8u;
    }
    const uint32_t item = a.first_item + w;
    const uint32_t tile = divide(item, a.by_span);
    const uint32_t span = item - tile * a.spans_per_tile;
    const uint32_t plane = divide(tile, a.by_pair);     // layer * 2 + kv
    const uint32_t i = tile - plane * a.pairs;
    const uint32_t layer = plane >> 1, kv = plane & 1u;

    const uint8_t *s;
    uint8_t *d;
    if (SRC == kPool) {
        s = reinterpret_cast<const uint8_t *>(table_entry(a.src_tab, kv * a.num_layers + layer)) +
            static_cast<uint64_t>(uniform(src_id<IDS>(a, i))) * a.tile_bytes;
    } else {
        const uint32_t x = IDS == kIdsDevice ? a.lin_first + i : uniform(src_id<IDS>(a, i));
        s = a.src_lin + (static_cast<uint64_t>(plane) * a.lin_pairs + x) * a.tile_bytes;
    }
    if (DST == kPool) {
        d = reinterpret_cast<uint8_t *>(table_entry(a.dst_tab, kv * a.num_layers + layer)) +
            static_cast<uint64_t>(uniform(dst_id<IDS>(a, i))) * a.tile_bytes;
    } else {
        d = a.dst_lin + (static_cast<uint64_t>(plane) * a.lin_pairs + a.lin_first + i) * a.tile_bytes;
    }

    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(s, a.tile_bytes);
    const __amdgpu_buffer_rsrc_t rd = tile_rsrc(d, a.tile_bytes);
    const uint32_t first = span * ROWS * kWaveRow, lane_off = (threadIdx.x % 64) * 16u;
    u32x4 r[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u)
        r[u] = buffer_load16(rs, row_offset(first + u * kWaveRow, a.tile_bytes) + lane_off);
#pragma unroll
    for (int u = 0; u < ROWS; ++u)
        buffer_store16(rd, row_offset(first + u * kWaveRow, a.tile_bytes) + lane_off, r[u]);
}

// Pool to pool, ids in the kernel arguments.
template <int IDS, int SPAN>
__global__ void __launch_bounds__(kThreads) copy_tiles(const CopyArgs a)
{
    const uint32_t lane_off = (threadIdx.x % 64) * 16u;
    const uint32_t waves = gridDim.x * (kThreads / 64);
    for (uint32_t w = blockIdx.x * (kThreads / 64) + threadIdx.x / 64; w < a.items; w += waves) {
        const uint32_t item = uniform(w);
        const uint32_t tile = item / a.spans_per_tile;
        const uint32_t span = item - tile * a.spans_per_tile;
        const uint32_t i = tile / a.planes;
        const uint32_t plane = tile - i * a.planes; // layer * 2 + kv
        const uint32_t layer = plane >> 1, kv = plane & 1u;
        const uint8_t *s = reinterpret_cast<const uint8_t *>(table_entry(a.src_tab, kv * a.num_layers + layer)) +
                           static_cast<uint64_t>(uniform(src_id<IDS>(a, i))) * a.tile_bytes;
        uint8_t *d = reinterpret_cast<uint8_t *>(table_entry(a.dst_tab, kv * a.num_layers + layer)) +
                     static_cast<uint64_t>(uniform(dst_id<IDS>(a, i))) * a.tile_bytes;

        const __amdgpu_buffer_rsrc_t rs = tile_rsrc(s, a.tile_bytes);
        const __amdgpu_buffer_rsrc_t rd = tile_rsrc(d, a.tile_bytes);
        const uint32_t first = span * SPAN * kWaveRow;
        u32x4 r[SPAN];
#pragma unroll
        for (int u = 0; u < SPAN; ++u)
            r[u] = buffer_load16(rs, row_offset(first + u * kWaveRow, a.tile_bytes) + lane_off);
#pragma unroll
        for (int u = 0; u < SPAN; ++u)
            buffer_store16(rd, row_offset(first + u * kWaveRow, a.tile_bytes) + lane_off, r[u]);
    }
}

uint32_t compute_units()
{
    static const uint32_t cus = [] {
        int dev = 0, n = 256;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            n = 256;
        return static_cast<uint32_t>(n);
    }();
    return cus;
}

// Span (in 1 KiB rows) for a bulk copy: the power of two nearest above a
// quarter of the tile, between 2 and 32.
int bulk_span(uint32_t tile_bytes)
{
    const uint32_t quarter = (tile_bytes + 4 * kWaveRow - 1) / (4 * kWaveRow);
    int span = 2;
    while (span < 32 && static_cast<uint32_t>(span) < quarter)
        span *= 2;
    return span;
}

template <int IDS>
const void *copy_kernel_span(int span)
{
    switch (span) {
    case 32:
        return reinterpret_cast<const void *>(&copy_tiles<IDS, 32>);
    case 16:
        return reinterpret_cast<const void *>(&copy_tiles<IDS, 16>);
    case 8:
        return reinterpret_cast<const void *>(&copy_tiles<IDS, 8>);
    case 4:
        return reinterpret_cast<const void *>(&copy_tiles<IDS, 4>);
    default:
        return reinterpret_cast<const void *>(&copy_tiles<IDS, 2>);
    }
}

template <int SRC, int DST, int IDS>
const void *copy_kernel_rows(int rows)
{
    return rows == 2 ? reinterpret_cast<const void *>(&copy_rows<SRC, DST, IDS, 2>)
                     : reinterpret_cast<const void *>(&copy_rows<SRC, DST, IDS, 1>);
}

template <int SRC, int DST>
const void *copy_kernel(int ids, int rows)
{
    if (ids == kIdsDevice)
        return copy_kernel_rows<SRC, DST, kIdsDevice>(rows);
    if (SRC == kPool && DST == kPool && ids == kIds16)
        return copy_kernel_rows<SRC, DST, kIds16>(rows);
    return copy_kernel_rows<SRC, DST, kIds32>(rows);
}

// Tiles from this size on are walked in runs of kXcdRun rows per XCD.
constexpr uint32_t kXcdRunTileBytes = 128u << 10;
// Resident wavefronts of a full CU; a launch of fewer rows than this per CU
// is small (a final stage).
constexpr uint32_t kWavesPerCU = 32;
// Capped launches: fewer wave items than this per CU take 2 KiB spans.
constexpr uint32_t kBulkWaveItemsPerCU = 16;
// Rows per launch: 64 lanes each, in 32-bit work-item counts.
constexpr uint32_t kMaxRowsPerLaunch = 1u << 24;
// max_workgroups > 0 caps the grid (pool to pool with host ids only): fewer,
// resident workgroups walk the items, leaving the rest of the chip (and of
// HBM) to other work.  ids16: every id of both lists is below 65536 (pool to
// pool only).  host_staging: the linear side is host memory.  Throws nothing.
template <int SRC, int DST>
int launch_copy(CopyArgs a, const int32_t *src_ids, const int32_t *dst_ids, int64_t n,
                bool ids_on_device, hipStream_t stream, uint32_t max_workgroups = 0, bool ids16 = false,
                const LaunchEvents &ev = LaunchEvents(), bool host_staging = false)
{
    const int ids = ids_on_device ? kIdsDevice : (SRC == kPool && DST == kPool && ids16) ? kIds16 : kIds32;
    const int64_t inline_pairs = ids == kIds16 ? 2 * kInlinePairs : kInlinePairs;
    const bool capped = SRC == kPool && DST == kPool && max_workgroups > 0 && !ids_on_device;
    const uint64_t pairs_first_launch = std::min<int64_t>(n, ids_on_device ? n : inline_pairs);
    const uint64_t planes = 2ull * a.num_layers;
    auto spans = [&](int kib) { return (a.tile_bytes + kib * kWaveRow - 1) / (kib * kWaveRow); };
    int span = 1;
    if (capped) {
        span = bulk_span(a.tile_bytes);
        if (pairs_first_launch * planes * spans(span) < kBulkWaveItemsPerCU * compute_units())
            span = 2;
    } else if (!host_staging && pairs_first_launch * planes * spans(1) <= kWavesPerCU * compute_units()) {
        span = 2;
    }
    a.spans_per_tile = spans(span);
    a.by_span = divisor(a.spans_per_tile);
    const uint64_t items_per_pair = planes * a.spans_per_tile;
    const uint64_t per_launch = std::min<uint64_t>(0x7fffffffull / items_per_pair,
                                                   ids_on_device ? UINT64_MAX : static_cast<uint64_t>(inline_pairs));
    if (per_launch == 0)
        return LLMIG_EINVAL;
    std::vector<uint64_t> ordered;
    if (!capped && DST == kPool && ids != kIdsDevice && ordering_pays(n, planes * a.tile_bytes)) {
        try {
            order_pairs(src_ids, dst_ids, n, ordered);
        } catch (...) {
            ordered.clear();    // no memory for it: the caller's order
        }
    }
    a.lin_pairs = static_cast<uint32_t>(n);
    a.planes = static_cast<uint32_t>(planes);
    a.xcd_runs = a.tile_bytes >= kXcdRunTileBytes ? 1u : 0u;
    const void *fn = !capped          ? copy_kernel<SRC, DST>(ids, span)
                     : ids == kIds16  ? copy_kernel_span<kIds16>(span)
                                      : copy_kernel_span<kIds32>(span);
    int64_t launch = 0;
    for (int64_t first = 0; first < n; first += static_cast<int64_t>(per_launch)) {
        const uint32_t m = static_cast<uint32_t>(std::min<int64_t>(n - first, per_launch));
        a.pairs = m;
        a.by_pair = divisor(m);
        a.lin_first = static_cast<uint32_t>(first);
        a.items = static_cast<uint32_t>(m * items_per_pair);
        if (ids == kIdsDevice) {
            a.src_ids_dev = src_ids ? src_ids + first : nullptr;
            a.dst_ids_dev = dst_ids ? dst_ids + first : nullptr;
        } else {
            inline_ids(a.ids, ids, src_ids, dst_ids, ordered, first, m);
        }
        void *args[] = {&a};
        const bool last_pairs = first + static_cast<int64_t>(per_launch) >= n;
        const uint32_t step = capped ? a.items : kMaxRowsPerLaunch;
        for (uint32_t at = 0; at < a.items; at += std::min(step, a.items - at)) {
            const uint32_t here = std::min(step, a.items - at);
            a.first_item = at;
            uint32_t grid = here / span, threads = 64u * span;  // here: a multiple of 2 for spans of 2
            if (capped) {
                grid = std::min({(here + kThreads / 64 - 1) / (kThreads / 64), kMaxGridWorkgroups, max_workgroups});
                threads = kThreads;
            }
            const bool last = last_pairs && at + here == a.items;
            hipError_t e = launch_kernel(fn, dim3(grid), dim3(threads), args, stream, ev, launch, last ? launch + 1 : -1);
            if (e != hipSuccess)
                return hip_error(e);
            ++launch;
        }
    }
    return LLMIG_OK;
}

} // namespace

// Cross-layout tile conversion: the stage copy between two pools that keep
// the (token, head, dim) elements of a tile in different orders.  Part of
// the single translation unit built from llmig.hip.
//
// What it computes: for every pair i, layer l and K/V, every element
// (t, h, d) of tile (l, kv) of source block src[i] lands in tile (l, kv) of
// destination block dst[i] at the position the destination's layout gives
// it (the layouts are listed with LLMIG_LAYOUT_* in llmig.h).  Whole tiles
// move, as in the same-layout copy (Llumnix §4.2), so a partial last block
// carries its unused slots along.
//
// Kernel design (CDNA4, wave64):
//  * In every layout a head's elements form one slab of block_size *
//    head_dim * 2 bytes: contiguous in HND, HCNX and HDN, and block_size
//    rows of head_dim * 2 bytes, one per token, in NHD.  A work item is one
//    (pair, layer, K/V, head) slab; it is read with 16-byte loads in the
//    source's own order (whole rows, coalesced) and written with 16-byte
//    stores in the destination's own order (contiguous), so neither side of
//    HBM sees a partial row.
//  * convert_slabs, every uncapped launch: one workgroup per slab, one
//    16-byte chunk per lane.  As in the same-layout copy, what bounds it is
//    HBM and the DRAM order of the bytes in flight, so each wavefront moves
//    1 KiB and the slabs run plane by plane over pairs ordered by destination
//    block (order_pairs).  Against the kernel below (a slab per wavefront, 4 chunks a lane,
//    pair by pair) on MI355X: 32 heads of 16 x 128, token-major to head-major
//    6.33 -> 6.75 TB/s, to HCNX/HDN 6.28 -> 6.68, back 6.04 -> 6.59; 8 heads
//    4.95 -> 6.49, 4.93 -> 6.15, 4.94 -> 6.30; one head 4.67 -> 6.06,
//    4.64 -> 5.63, 4.63 -> 5.78.
//  * Each XCD takes runs of kSlabRun = 64 slabs, so that the slabs of one
//    token-major tile, which share its rows, meet in one L2.  32 heads,
//    token-major to head-major: dealt in turn 6.12, runs of 16 6.56, 64
//    6.75, 256 6.68, 1024 6.70 TB/s; 8 heads 6.12, 6.14, 6.49, 6.24, 6.38.
//  * Between reading and writing the slab passes through LDS, which is where
//    the layouts transpose.  A 16-byte chunk is 8 consecutive dims of one
//    token in NHD, HND and HCNX, and 8 consecutive tokens of one dim in HDN.
//    Between the first three a chunk moves whole (one ds_read_b128 per
//    chunk); to or from HDN every output chunk gathers 8 16-bit elements
//    from 8 source chunks.  The LDS image has one 16-byte pad after every 16
//    chunks, which spreads the strided reads of both cases over distinct
//    banks for the common shapes (block_size 16, head_dim 64 or 128).
//  * A plane whose two layouts agree (say K converts and V does not) moves
//    chunk for chunk, registers straight to the store, without LDS; so does,
//    in convert_slabs, one between NHD and HND, whose slabs hold their chunks
//    in one order.
//  * convert_tiles, launches under a workgroup cap (the throttle of a
//    migration's non-final stages): few resident workgroups, so each
//    wavefront keeps a whole slab in flight.  Two wavefronts per workgroup
//    (two adjacent heads of one tile): 8% faster than four when the source
//    is token-major, equal the other way.  Consecutive workgroups share an
//    XCD.
//  * Index arithmetic divides chunk numbers (< 2^16) by per-call constants
//    with a multiply-high by ceil(2^32 / divisor), exact in that range.
//  * Block ids, layouts and base addresses are wavefront-uniform and come
//    from the kernel arguments or scalar loads; ids travel inline as in the
//    same-layout copy (512 pairs of packed 16-bit ids a launch when both
//    pools have at most 65536 blocks, else 256 pairs of 32-bit ids).
//  * Global accesses are raw buffer loads and stores over one tile with the
//    same cache policy as the same-layout copy (nt loads, sc1 nt stores).
//  * The source may also be a staging buffer laid out as llmig_pack writes
//    it (the receiving side of block fusion, §5, converting as it scatters).
#pragma once

#include <algorithm>
#include <cstring>
#include <vector>

#include "common.h"

namespace {

constexpr int kMaxSlabChunksPerLane = 16;           // slabs of up to 16 KiB
constexpr int kConvertWaves = 2;                    // wavefronts per workgroup
constexpr uint32_t kXcds = 8;                       // accelerator dies the dispatcher deals workgroups to
constexpr uint32_t kSlabRun = 64;                   // convert_slabs: slabs in a row on one XCD

// What a launch moves between which layouts, without its block ids.
struct ConvertShape {
    const uint64_t *src_tab;
    const uint64_t *dst_tab;
    const uint8_t *src_lin;     // staging buffer [L][2][lin_pairs][tile] (null: source is a pool)
    const int32_t *src_ids_dev; // device id lists (null when the ids are inline)
    const int32_t *dst_ids_dev;
    uint64_t magic_row;         // ceil(2^32 / row_chunks)
    uint64_t magic_bs;          // ceil(2^32 / block_size)
    uint64_t magic_t;           // ceil(2^32 / t_chunks)
    uint32_t tile_bytes;
    uint32_t num_layers;
    uint32_t heads;
    uint32_t block_size;
    uint32_t row_chunks;        // head_dim / 8: chunks of one token's head
    uint32_t t_chunks;          // block_size / 8: chunks of one dim's tokens (HDN)
    uint32_t chunks;            // chunks of one head slab
    uint32_t pairs;             // pairs in this launch
    uint32_t units;             // slabs: pairs * 2 * num_layers * heads
    uint32_t first_unit;        // this launch's first slab (convert_slabs)
    Divisor by_head, by_pair;   // division by heads and by pairs (not convert_tiles)
    uint32_t lin_first;         // this launch's first pair within the whole call
    uint32_t lin_pairs;         // pairs in the whole call (plane stride of the staging buffer)
    uint32_t first_slot;        // write_slabs: slot of the launch's first token in its block
    uint32_t tokens;            // write_slabs: tokens in this launch
    int32_t layouts[4];         // source K, source V, destination K, destination V
};

struct ConvertArgs : ConvertShape {
    uint32_t ids[2 * kInlinePairs]; // inline ids, laid out as the launch's Ids mode says
};

// A write lists one block per id; its arguments are half as long (they are
// copied into the launch: 16 writes of 7 tokens 133.3 -> 131.8 us).
struct SlabWriteArgs : ConvertShape {
    uint32_t ids[kInlinePairs];
};

__device__ __forceinline__ uint32_t div_magic(uint32_t n, uint64_t magic)
{
    return static_cast<uint32_t>((static_cast<uint64_t>(n) * magic) >> 32);
}

// Byte offset inside a tile of chunk k (in the layout's own order) of head h.
__device__ __forceinline__ uint32_t slab_offset(int32_t layout, uint32_t h, uint32_t k, const ConvertShape &a)
{
    if (layout == LLMIG_LAYOUT_NHD) {
        const uint32_t t = div_magic(k, a.magic_row);
        const uint32_t c = k - t * a.row_chunks;
        return ((t * a.heads + h) * a.row_chunks + c) * 16u;
    }
    return (h * a.chunks + k) * 16u;
}

// Slab index of the chunk holding dims [8c, 8c + 8) of token t, in a layout
// whose chunks run along the dims (NHD, HND, HCNX).
__device__ __forceinline__ uint32_t dim_chunk_index(int32_t layout, uint32_t t, uint32_t c, const ConvertShape &a)
{
    return layout == LLMIG_LAYOUT_HCNX ? c * a.block_size + t : t * a.row_chunks + c;
}

__device__ __forceinline__ uint32_t padded(uint32_t k)
{
    return k + (k >> 4);
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int IDS>
__device__ __forceinline__ uint32_t convert_src_id(const ConvertArgs &a, uint32_t i)
{
    if (IDS == kIds16)
        return a.ids[i] & 0xffffu;
    return IDS == kIds32 ? a.ids[i] : static_cast<uint32_t>(id_entry(a.src_ids_dev, i));
}

template <int IDS>
__device__ __forceinline__ uint32_t convert_dst_id(const ConvertArgs &a, uint32_t i)
{
    if (IDS == kIds16)
        return a.ids[i] >> 16;
    return IDS == kIds32 ? a.ids[kInlinePairs + i] : static_cast<uint32_t>(id_entry(a.dst_ids_dev, i));
}

// Element e of the eight chunks first, first + step, ... of a padded slab.
// (The loop adds: with a multiplication per element the index arithmetic,
// not HBM, bounded the conversions to HDN: 32 heads of 16 x 128, token-major
// to HDN 6.14 TB/s, now 6.44.)
__device__ __forceinline__ u32x4 gather8(const u32x4 *slab, uint32_t first, uint32_t step, uint32_t e)
{
    const uint16_t *slab16 = reinterpret_cast<const uint16_t *>(slab) + e;
    uint32_t x[8], at = first;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        x[j] = slab16[padded(at) * 8u];
        at += step;
    }
    return u32x4{x[0] | (x[1] << 16), x[2] | (x[3] << 16), x[4] | (x[5] << 16), x[6] | (x[7] << 16)};
}

// Output chunk k of a slab, gathered from the slab's padded LDS image (in the
// source's chunk order).
__device__ __forceinline__ u32x4 gather_chunk(const u32x4 *slab, uint32_t k, int32_t sl, int32_t dl,
                                              const ConvertShape &a)
{
    if (dl == LLMIG_LAYOUT_HDN) {
        // tokens [8 tg, 8 tg + 8) of dim dd
        const uint32_t dd = div_magic(k, a.magic_t);
        const uint32_t tg = k - dd * a.t_chunks;
        const uint32_t c = dd >> 3, e = dd & 7u;
        // tokens of a dim: row_chunks apart (NHD, HND) or next to each other
        const uint32_t step = sl == LLMIG_LAYOUT_HCNX ? 1u : a.row_chunks;
        return gather8(slab, dim_chunk_index(sl, 8u * tg, c, a), step, e);
    }
    // dims [8 c, 8 c + 8) of token t
    uint32_t t, c;
    if (dl == LLMIG_LAYOUT_HCNX) {
        c = div_magic(k, a.magic_bs);
        t = k - c * a.block_size;
    } else {
        t = div_magic(k, a.magic_row);
        c = k - t * a.row_chunks;
    }
    if (sl == LLMIG_LAYOUT_HDN) {
        const uint32_t tg = t >> 3, e = t & 7u;
        return gather8(slab, 8u * c * a.t_chunks + tg, a.t_chunks, e);
    }
    return slab[padded(dim_chunk_index(sl, t, c, a))];
}

// Slab of workgroup w (kSlabRun consecutive slabs on one XCD; the dispatcher
// hands workgroup g to XCD g % 8; the grid's tail keeps its order).
__device__ __forceinline__ uint32_t slab_of(uint32_t w)
{
    const uint32_t round = w / (kXcds * kSlabRun), r8 = w % (kXcds * kSlabRun);
    if ((round + 1u) * (kXcds * kSlabRun) <= gridDim.x)
        w = round * (kXcds * kSlabRun) + (r8 % kXcds) * kSlabRun + r8 / kXcds;
    return w;
}

// One workgroup per slab, one 16-byte chunk per lane (WAVES wavefronts cover
// the slab; the launch leaves out those past its end).
template <int IDS, int WAVES>
__global__ void __launch_bounds__(WAVES * 64) convert_slabs(const ConvertArgs a)
{
    __shared__ u32x4 lds[68 * WAVES];                // 64 WAVES chunks + one pad per 16
    const uint32_t k = threadIdx.x;
    const uint32_t unit = a.first_unit + slab_of(blockIdx.x);
    const uint32_t tile = divide(unit, a.by_head);
    const uint32_t h = unit - tile * a.heads;
    const uint32_t plane = divide(tile, a.by_pair);
    const uint32_t i = tile - plane * a.pairs;
    const uint32_t layer = plane >> 1, kv = plane & 1u;
    const int32_t sl = a.layouts[kv], dl = a.layouts[2 + kv];

    const uint8_t *s;
    if (a.src_lin) {
        const uint32_t x = IDS == kIdsDevice ? a.lin_first + i : uniform(convert_src_id<IDS>(a, i));
        s = a.src_lin + (static_cast<uint64_t>(plane) * a.lin_pairs + x) * a.tile_bytes;
    } else {
        s = reinterpret_cast<const uint8_t *>(table_entry(a.src_tab, kv * a.num_layers + layer)) +
            static_cast<uint64_t>(uniform(convert_src_id<IDS>(a, i))) * a.tile_bytes;
    }
    uint8_t *d = reinterpret_cast<uint8_t *>(table_entry(a.dst_tab, kv * a.num_layers + layer)) +
                 static_cast<uint64_t>(uniform(convert_dst_id<IDS>(a, i))) * a.tile_bytes;
    // lanes past the slab: out of the resource's range, loads 0 and stores nothing
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(s, a.tile_bytes);
    const __amdgpu_buffer_rsrc_t rd = tile_rsrc(d, a.tile_bytes);
    const bool in = k < a.chunks;
    const u32x4 r = buffer_load16(rs, in ? slab_offset(sl, h, k, a) : kOutOfRange);
    const uint32_t to = in ? slab_offset(dl, h, k, a) : kOutOfRange;
    // NHD and HND hold a slab's chunks in one order (token by token): only
    // the place of its rows in the tile differs
    if (sl == dl || (sl <= LLMIG_LAYOUT_HND && dl <= LLMIG_LAYOUT_HND)) {
        buffer_store16(rd, to, r);
        return;
    }
    lds[padded(k)] = r;
    __syncthreads();
    if (in)
        buffer_store16(rd, to, gather_chunk(lds, k, sl, dl, a));
}

// Token writes: the slab of one head of the launch's block i receives the
// tokens that data (a.src_lin, [L][K,V][a.lin_pairs tokens][heads][head_dim])
// holds of that block: slots [lo, hi).  As convert_slabs from a token-major
// source, with what lies outside those slots left alone: a chunk is one
// token's in NHD, HND and HCNX; in HDN it is 8 tokens' and is stored element
// by element where not all 8 are written.
template <int WAVES>
__global__ void __launch_bounds__(WAVES * 64) write_slabs(const SlabWriteArgs a)
{
    __shared__ u32x4 lds[68 * WAVES];
    const uint32_t k = threadIdx.x;
    const uint32_t unit = a.first_unit + slab_of(blockIdx.x);
    const uint32_t tile = divide(unit, a.by_head);
    const uint32_t h = unit - tile * a.heads;
    const uint32_t plane = divide(tile, a.by_pair);
    const uint32_t i = tile - plane * a.pairs;
    const uint32_t layer = plane >> 1, kv = plane & 1u;
    const int32_t dl = a.layouts[2 + kv];
    const uint32_t lo = i == 0 ? a.first_slot : 0u;
    const uint32_t hi = min(a.block_size, a.first_slot + a.tokens - i * a.block_size);
    // the row that slot 0 of the block would have in data (slots before lo are not read)
    const uint8_t *s = a.src_lin + ((static_cast<uint64_t>(plane) * a.lin_pairs + a.lin_first) * a.heads + h) *
                                       (a.row_chunks * 16u) +
                       (static_cast<int64_t>(i) * a.block_size - a.first_slot) *
                           static_cast<int64_t>(a.heads * a.row_chunks * 16u);
    uint8_t *d = reinterpret_cast<uint8_t *>(table_entry(a.dst_tab, kv * a.num_layers + layer)) +
                 static_cast<uint64_t>(uniform(a.ids[i])) * a.tile_bytes;
    const __amdgpu_buffer_rsrc_t rd = tile_rsrc(d, a.tile_bytes);
    const uint32_t t = div_magic(k, a.magic_row);
    const bool in = k < a.chunks && t >= lo && t < hi;
    u32x4 r = {0u, 0u, 0u, 0u};
    if (in)
        r = load16(s + slab_offset(LLMIG_LAYOUT_NHD, 0, k, a));
    if (dl <= LLMIG_LAYOUT_HND) {
        buffer_store16(rd, in ? slab_offset(dl, h, k, a) : kOutOfRange, r);
        return;
    }
    lds[padded(k)] = r;
    __syncthreads();
    if (k >= a.chunks)
        return;
    const uint32_t to = slab_offset(dl, h, k, a);
    const u32x4 v = gather_chunk(lds, k, LLMIG_LAYOUT_NHD, dl, a);
    if (dl == LLMIG_LAYOUT_HCNX) {
        const uint32_t slot = k - div_magic(k, a.magic_bs) * a.block_size;
        buffer_store16(rd, slot >= lo && slot < hi ? to : kOutOfRange, v);
        return;
    }
    const uint32_t t0 = 8u * (k - div_magic(k, a.magic_t) * a.t_chunks);
    if (t0 >= lo && t0 + 8u <= hi) {
        buffer_store16(rd, to, v);
        return;
    }
    const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (uint32_t e = 0; e < 8; ++e)
        if (t0 + e >= lo && t0 + e < hi)
            *(LLMIG_GLOBAL uint16_t *)(d + to + 2u * e) = static_cast<uint16_t>(w4[e / 2] >> (16u * (e & 1u)));
}

// A capped grid: kConvertWaves wavefronts walk the slabs, N chunks per lane.
template <int IDS, int N>
__global__ void __launch_bounds__(kConvertWaves * 64) convert_tiles(const ConvertArgs a)
{
    __shared__ u32x4 lds[kConvertWaves][68 * N];     // 64 N chunks + one pad per 16
    const uint32_t lane = threadIdx.x % 64;
    const uint32_t wave = threadIdx.x / 64;
    u32x4 *mine = lds[wave];
    const uint32_t waves = gridDim.x * kConvertWaves;
    const uint32_t per_pair_plane = a.heads;
    const uint32_t planes = 2u * a.num_layers;

    // consecutive workgroups (the heads of one tile) on one XCD
    const uint32_t full = gridDim.x - gridDim.x % kXcds;
    const uint32_t group = blockIdx.x < full ? (blockIdx.x % kXcds) * (full / kXcds) + blockIdx.x / kXcds
                                             : blockIdx.x;
    for (uint32_t w = group * kConvertWaves + wave; w < a.units; w += waves) {
        const uint32_t unit = uniform(w);
        const uint32_t tile = unit / per_pair_plane;
        const uint32_t h = unit - tile * per_pair_plane;
        const uint32_t i = tile / planes;
        const uint32_t plane = tile - i * planes;
        const uint32_t layer = plane >> 1, kv = plane & 1u;
        const int32_t sl = a.layouts[kv], dl = a.layouts[2 + kv];

        const uint8_t *s;
        s = reinterpret_cast<const uint8_t *>(table_entry(a.src_tab, kv * a.num_layers + layer)) +
            static_cast<uint64_t>(uniform(convert_src_id<IDS>(a, i))) * a.tile_bytes;
        uint8_t *d = reinterpret_cast<uint8_t *>(table_entry(a.dst_tab, kv * a.num_layers + layer)) +
                     static_cast<uint64_t>(uniform(convert_dst_id<IDS>(a, i))) * a.tile_bytes;
        const __amdgpu_buffer_rsrc_t rs = tile_rsrc(s, a.tile_bytes);
        const __amdgpu_buffer_rsrc_t rd = tile_rsrc(d, a.tile_bytes);

        u32x4 r[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const uint32_t k = lane + 64u * u;
            if (k < a.chunks)
                r[u] = buffer_load16(rs, slab_offset(sl, h, k, a));
        }
        if (sl == dl) {
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const uint32_t k = lane + 64u * u;
                if (k < a.chunks)
                    buffer_store16(rd, slab_offset(dl, h, k, a), r[u]);
            }
            continue;
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const uint32_t k = lane + 64u * u;
            if (k < a.chunks)
                mine[padded(k)] = r[u];
        }
        wave_lds_sync();
        // Output chunks: fully unrolled for small slabs; for large ones two at
        // a time, which keeps the gathers' registers within four waves' share.
        constexpr int kGatherUnroll = N > 4 ? 2 : N;
#pragma unroll kGatherUnroll
        for (int u = 0; u < N; ++u) {
            const uint32_t k = lane + 64u * u;
            if (k >= a.chunks)
                continue;
            buffer_store16(rd, slab_offset(dl, h, k, a), gather_chunk(mine, k, sl, dl, a));
        }
        wave_lds_sync();
    }
}

template <int IDS>
const void *convert_kernel_n(int n)
{
    switch (n) {
    case 16:
        return reinterpret_cast<const void *>(&convert_tiles<IDS, 16>);
    case 8:
        return reinterpret_cast<const void *>(&convert_tiles<IDS, 8>);
    case 4:
        return reinterpret_cast<const void *>(&convert_tiles<IDS, 4>);
    case 2:
        return reinterpret_cast<const void *>(&convert_tiles<IDS, 2>);
    default:
        return reinterpret_cast<const void *>(&convert_tiles<IDS, 1>);
    }
}

template <int IDS>
const void *convert_kernel_waves(int waves)
{
    switch (waves) {
    case 16:
        return reinterpret_cast<const void *>(&convert_slabs<IDS, 16>);
    case 8:
        return reinterpret_cast<const void *>(&convert_slabs<IDS, 8>);
    case 4:
        return reinterpret_cast<const void *>(&convert_slabs<IDS, 4>);
    case 2:
        return reinterpret_cast<const void *>(&convert_slabs<IDS, 2>);
    default:
        return reinterpret_cast<const void *>(&convert_slabs<IDS, 1>);
    }
}

const void *write_kernel(int waves)
{
    switch (waves) {
    case 16:
        return reinterpret_cast<const void *>(&write_slabs<16>);
    case 8:
        return reinterpret_cast<const void *>(&write_slabs<8>);
    case 4:
        return reinterpret_cast<const void *>(&write_slabs<4>);
    case 2:
        return reinterpret_cast<const void *>(&write_slabs<2>);
    default:
        return reinterpret_cast<const void *>(&write_slabs<1>);
    }
}

const void *convert_kernel(int ids, int n, bool capped)
{
    if (capped)
        return ids == kIds16 ? convert_kernel_n<kIds16>(n) : convert_kernel_n<kIds32>(n);
    if (ids == kIdsDevice)
        return convert_kernel_waves<kIdsDevice>(n);
    return ids == kIds16 ? convert_kernel_waves<kIds16>(n) : convert_kernel_waves<kIds32>(n);
}

uint64_t magic_for(uint32_t divisor)
{
    return ((1ull << 32) + divisor - 1) / divisor;
}

void convert_magic(ConvertShape &a)
{
    a.magic_row = magic_for(a.row_chunks);
    a.magic_bs = magic_for(a.block_size);
    a.magic_t = magic_for(a.t_chunks > 0 ? a.t_chunks : 1u);
    a.by_head = divisor(a.heads);
}

// Chunks per lane (a power of two) for slabs of `chunks` 16-byte chunks.
int convert_chunks_per_lane(uint32_t chunks)
{
    int n = 1;
    while (static_cast<uint32_t>(n) * 64u < chunks)
        n *= 2;
    return n;
}

// Launches the conversion of n pairs (src_ids null: the source is the staging
// buffer a.src_lin, one tile per pair and plane).  The caller has checked
// that the geometry is supported (16-bit elements, head_dim % 8 == 0,
// block_size % 8 == 0 when a side is HDN, slabs of at most 16 KiB).
// ids16: every id of both lists is below 65536 (pool to pool only).
// max_workgroups > 0 (pool to pool with host ids only) caps the grid.
int launch_convert(ConvertArgs a, const int32_t *src_ids, const int32_t *dst_ids, int64_t n, bool ids_on_device,
                   hipStream_t stream, uint32_t max_workgroups, const LaunchEvents &ev = LaunchEvents(),
                   bool ids16 = false)
{
    const int ids = ids_on_device ? kIdsDevice : (src_ids && ids16) ? kIds16 : kIds32;
    const uint64_t inline_pairs = ids == kIds16 ? 2 * kInlinePairs : kInlinePairs;
    const bool capped = max_workgroups > 0 && src_ids && !ids_on_device;
    const int per_lane = convert_chunks_per_lane(a.chunks);
    if (per_lane > kMaxSlabChunksPerLane)
        return LLMIG_EINVAL;
    convert_magic(a);
    const uint64_t units_per_pair = 2ull * a.num_layers * a.heads;
    const uint64_t per_launch = std::min<uint64_t>(0x7fffffffull / units_per_pair,
                                                   ids_on_device ? UINT64_MAX : inline_pairs);
    if (per_launch == 0)
        return LLMIG_EINVAL;
    std::vector<uint64_t> ordered;
    if (!capped && !ids_on_device && ordering_pays(n, 2ull * a.num_layers * a.tile_bytes)) {
        try {
            order_pairs(src_ids, dst_ids, n, ordered);
        } catch (...) {
            ordered.clear();    // no memory for it: the caller's order
        }
    }
    const void *fn = convert_kernel(ids, per_lane, capped);
    const uint32_t threads = capped ? kConvertWaves * 64u : (a.chunks + 63u) / 64u * 64u;
    // work-items of a launch are counted in 32 bits
    const uint32_t step = capped ? 0x7fffffffu : (1u << 30) / threads;
    a.lin_pairs = static_cast<uint32_t>(n);
    int64_t launch = 0;
    for (int64_t first = 0; first < n; first += static_cast<int64_t>(per_launch)) {
        const uint32_t m = static_cast<uint32_t>(std::min<int64_t>(n - first, per_launch));
        a.pairs = m;
        a.by_pair = divisor(m);
        a.units = static_cast<uint32_t>(m * units_per_pair);
        a.lin_first = static_cast<uint32_t>(first);
        if (ids == kIdsDevice) {
            a.src_ids_dev = src_ids ? src_ids + first : nullptr;
            a.dst_ids_dev = dst_ids + first;
        } else {
            inline_ids(a.ids, ids, src_ids, dst_ids, ordered, first, m);
        }
        void *args[] = {&a};
        const bool last_pairs = first + static_cast<int64_t>(per_launch) >= n;
        for (uint32_t at = 0; at < a.units; at += std::min(step, a.units - at)) {
            const uint32_t here = std::min(step, a.units - at);
            a.first_unit = at;
            const uint32_t grid = capped ? std::min({(here + kConvertWaves - 1) / kConvertWaves, kMaxGridWorkgroups,
                                                     max_workgroups})
                                         : here;
            const bool last = last_pairs && at + here == a.units;
            hipError_t e = launch_kernel(fn, dim3(grid), dim3(threads), args, stream, ev, launch, last ? launch + 1 : -1);
            if (e != hipSuccess)
                return hip_error(e);
            ++launch;
        }
    }
    return LLMIG_OK;
}

} // namespace

// Shared definitions of the llmig kernels: launch geometry, the 16-byte
// word type, address-space helpers and the library's HIP error record.
// Part of the single translation unit built from llmig.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <vector>

#include "llmig.h"

namespace {

constexpr int kThreads = 256;                 // 4 wavefronts of 64 lanes
constexpr uint32_t kRowBytes = kThreads * 16; // one 16-byte word per lane of a workgroup
constexpr int kInlinePairs = 256;             // ids carried in the kernel arguments per launch
// Grid cap of the grid-stride kernels (copy, conversion, token writes): a
// dispatch counts its work-items in 32 bits, and past a few million
// workgroups more of them would only wait in the queue.
constexpr uint32_t kMaxGridWorkgroups = 1u << 22;

// Where a launch finds its block ids.
enum Ids {
    kIdsDevice = 0, // device arrays src_ids_dev / dst_ids_dev
    kIds32 = 1,     // ids[i] (source) and ids[kInlinePairs + i] (destination)
    kIds16 = 2,     // ids[i] = source | destination << 16 (pool to pool, ids below 65536)
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

thread_local int g_last_hip_error = 0;

int hip_error(hipError_t e)
{
    g_last_hip_error = static_cast<int>(e);
    return LLMIG_EHIP;
}

// Optional events around a call's kernels: start is recorded on the stream
// right before the first kernel is launched and stop right after the last
// one, so their interval holds the kernels (and one launch's latency) but
// none of the host work that planned them.
struct LaunchEvents {
    hipEvent_t start = nullptr;
    hipEvent_t stop = nullptr;
};

// Launch k of `launches` of one call (launches -1: not the last one).
hipError_t launch_kernel(const void *fn, dim3 grid, dim3 block, void **args, hipStream_t stream,
                         const LaunchEvents &ev, int64_t k, int64_t launches)
{
    hipError_t e = hipSuccess;
    if (k == 0 && ev.start)
        e = hipEventRecord(ev.start, stream);
    if (e == hipSuccess)
        e = hipLaunchKernel(fn, grid, block, args, 0, stream);
    if (e == hipSuccess && k == launches - 1 && ev.stop)
        e = hipEventRecord(ev.stop, stream);
    return e;
}

// Address spaces: global for the copied bytes (global_load/global_store
// instead of flat), constant for the small read-only tables so uniform
// reads of them become scalar loads.
#define LLMIG_GLOBAL __attribute__((address_space(1)))
#define LLMIG_CONSTANT __attribute__((address_space(4)))

__device__ __forceinline__ uint32_t uniform(uint32_t x)
{
    return __builtin_amdgcn_readfirstlane(x);
}

// Division of n < 2^31 by a per-call constant (Granlund and Montgomery 1994):
// with 2^(s-1) < d <= 2^s and m = ceil(2^(31 + s) / d), n / d is the high word
// of n * m shifted right by s - 1.  On a uniform n these are three scalar
// instructions, where the compiler's division by an unknown number is some
// twenty dependent vector ones, which shows with 1 KiB of work per wavefront
// (copy_tiles.h): 256 pairs of 128 KiB tiles to HCNX/HDN 655 -> 643 us, a
// prompt of 2000 tokens into them 326 -> 320; the copy itself +0.1%.
struct Divisor {
    uint32_t d, m, shift;
};

inline Divisor divisor(uint32_t d)
{
    uint32_t s = 0;
    while ((1ull << s) < d)
        ++s;
    if (s == 0)
        return Divisor{d, 0u, 0u};      // by 1
    return Divisor{d, static_cast<uint32_t>(((1ull << (31 + s)) + d - 1) / d), s - 1};
}

__device__ __forceinline__ uint32_t divide(uint32_t n, const Divisor &v)
{
    return v.d == 1u ? n : __umulhi(n, v.m) >> v.shift;
}

__device__ __forceinline__ uint64_t table_entry(const uint64_t *tab, uint32_t k)
{
    return ((const LLMIG_CONSTANT uint64_t *)tab)[k]; // address-space cast
}

__device__ __forceinline__ int32_t id_entry(const int32_t *ids, uint32_t k)
{
    return ((const LLMIG_CONSTANT int32_t *)ids)[k];
}

__device__ __forceinline__ u32x4 load16(const uint8_t *p)
{
    return __builtin_nontemporal_load((const LLMIG_GLOBAL u32x4 *)p);
}

__device__ __forceinline__ void store16(uint8_t *p, u32x4 v)
{
    __builtin_nontemporal_store(v, (LLMIG_GLOBAL u32x4 *)p);
}

// Raw buffer accesses (the migration copy): a resource over one tile, and
// 16-byte loads and stores with explicit cache-policy bits.  On gfx950 the
// policy bits are sc0 = 1, nt = 2, sc1 = 16 (sc1 alone selects device
// scope).  Loads stream (nt); stores also carry sc1, measured 0.5-1.3%
// faster on the LLaMA-7B stage than nt alone (plain or sc0 stores were
// 2-10% slower).  An access whose offset lies past the resource's
// num_records is out of range: a load returns zeros and a store is dropped.
// Tiles are at most 2^31 - 1 bytes, so kOutOfRange plus a lane's offset is
// always past a tile's resource.
constexpr uint32_t kOutOfRange = 0x80000000u;
constexpr int kBufferWord3 = 0x00020000;     // descriptor word 3 for raw 32-bit accesses on gfx9
constexpr int kStreamLoad = 2;               // nt
constexpr int kStreamStore = 16 | 2;         // sc1 nt

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const uint8_t *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base), 0, static_cast<int>(bytes), kBufferWord3);
}

__device__ __forceinline__ u32x4 buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kStreamLoad));
}

__device__ __forceinline__ void buffer_store16(__amdgpu_buffer_rsrc_t r, uint32_t off, u32x4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, kStreamStore);
}

// Whether a copy of n pairs of pair_bytes bytes each (one way, all layers, K
// and V) is worth ordering by destination on the host before its first launch.
// Ordering takes 2-4 ns a pair and delays that launch, so the copy of a pair
// must take longer, 20 ns from 64 KiB on; and the call must be longer than
// the queue of one launch, or DRAM has no order to see.  Measured, read +
// written: 24 MB of 366 pairs 10.6 us in the caller's order, 11.7 ordered; 48
// MB of 183 10.5 and 11.3; 64 MB level; 96 MB of 732 22.0 and 21.0; 170 MB of
// 400 29.8 and 28.2; 16 KiB a pair, 12000 pairs level, and up to 13% slower
// where the call has the GPU to itself; 64 KiB a pair, 12000 pairs 368 and 320.
constexpr int64_t kSortPairs = 32;
constexpr uint64_t kSortPairBytes = 64 << 10, kSortCallBytes = 48 << 20;

inline bool ordering_pays(int64_t n, uint64_t pair_bytes)
{
    return n >= kSortPairs && pair_bytes >= kSortPairBytes &&
           static_cast<uint64_t>(n) >= (kSortCallBytes + pair_bytes - 1) / pair_bytes;
}

// Orders the pairs of a call by the leading 11 bits of their destination ids
// (of the largest one's bits): out[k] = (source, destination) as one word,
// source in the low half.  src null: the source of pair k is k.  One counting
// pass, as fast to copy in as a full sort (which took two or three), and
// 5-10% sooner enqueued for calls of thousands of pairs.
void order_pairs(const int32_t *src, const int32_t *dst, int64_t n, std::vector<uint64_t> &out)
{
    constexpr int kBits = 11;
    out.resize(static_cast<size_t>(n));
    uint32_t all = 0;
    for (int64_t k = 0; k < n; ++k)
        all |= static_cast<uint32_t>(dst[k]);
    int shift = 0;
    while ((all >> shift) >> kBits)
        ++shift;
    uint32_t at[1u << kBits] = {};
    for (int64_t k = 0; k < n; ++k)
        ++at[static_cast<uint32_t>(dst[k]) >> shift];
    uint32_t sum = 0;
    for (uint32_t &c : at) {
        const uint32_t here = c;
        c = sum;
        sum += here;
    }
    for (int64_t k = 0; k < n; ++k) {
        const uint32_t d = static_cast<uint32_t>(dst[k]);
        out[at[d >> shift]++] = static_cast<uint64_t>(d) << 32 | static_cast<uint32_t>(src ? src[k] : static_cast<int32_t>(k));
    }
}

// Puts pairs [first, first + m) of a call into a launch's inline ids.  src
// null (a staging source): the pair's place in the call takes its place;
// dst null (a staging destination): none.  A call of thousands of pairs of
// small tiles is a chain of launches as short as this code (2000 pairs of 4
// KiB through a staging buffer: 16 launches in 68 us, 71 with a branch for
// every id), so each case is a copy or a plain loop.
inline void inline_ids(uint32_t *ids, int mode, const int32_t *src, const int32_t *dst,
                       const std::vector<uint64_t> &ordered, int64_t first, uint32_t m)
{
    if (!ordered.empty()) {
        const uint64_t *p = ordered.data() + first;
        for (uint32_t k = 0; k < m; ++k) {
            const uint32_t s = static_cast<uint32_t>(p[k]), d = static_cast<uint32_t>(p[k] >> 32);
            ids[k] = mode == kIds16 ? s | d << 16 : s;
            if (mode != kIds16)
                ids[kInlinePairs + k] = d;
        }
    } else if (mode == kIds16) {
        for (uint32_t k = 0; k < m; ++k)
            ids[k] = static_cast<uint32_t>(src[first + k]) | static_cast<uint32_t>(dst[first + k]) << 16;
    } else {
        if (src)
            std::memcpy(ids, src + first, m * sizeof(int32_t));
        else
            for (uint32_t k = 0; k < m; ++k)
                ids[k] = static_cast<uint32_t>(first) + k;
        if (dst)
            std::memcpy(ids + kInlinePairs, dst + first, m * sizeof(int32_t));
    }
}

} // namespace

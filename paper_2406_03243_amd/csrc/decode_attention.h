// Paged decode attention: the decode work that runs beside a migration and
// whose slowdown Llumnix §6.2 measures.  Part of the single translation unit
// built from llmig.hip.
//
// For layer l, sequence b and query head h (KV head g = h / group):
//     out[l][b][h] = softmax_t(scale * q[l][b][h] . K_l[t][g]) . V_l[t][g]
// over the sequence's ctx tokens, reached through its block table; inputs
// are fp16 or bf16, accumulation and output fp32.
//
// Layout of the work: sequences are cut into partitions of at most
// kPartTokens tokens (flash-decoding), so a long request does not leave one
// workgroup working alone; a workgroup takes one (partition, layer, KV head)
// and its four wavefronts take alternate 16-token groups of the partition; a
// second kernel merges the partitions of each sequence of more than one (a
// sequence of one partition is finished by its workgroup).  With `group`
// query heads per KV head, every K/V byte feeds `group` multiply-adds, a
// small dense contraction that runs on the matrix cores (see
// attn_partial_mfma).
#pragma once

#include <algorithm>

#include "common.h"

namespace {

#define LLMIG_LDS __attribute__((address_space(3)))

// s_waitcnt immediates (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt
// in 6:4, lgkmcnt in 11:8; a field at its maximum does not wait): until every
// vector-memory load has returned, and until every LDS access has.
constexpr int kWaitVm0 = 0x0F70;
constexpr int kWaitLgkm0 = 0xC07F;

constexpr int kPartTokens = 2048;    // most tokens per partition
constexpr int kMinPartTokens = 256;  // fewest tokens a sequence is split down to
constexpr int kWholeTokens = 768;    // a call of no longer sequences splits none
constexpr int kAttnMaxBatch = 256;   // sequences per call (their partitions ride in the kernel arguments)
// A partial result record: the partition's maximum score m (natural base),
// its weight sum l, two floats of padding, then the D weighted V sums, so
// that records (D + kAttnHeader floats) and their sums start on 16 bytes.
constexpr int kAttnHeader = 4;

// The sequences of a call in launch order: those cut into several partitions
// first, then those of one partition, each longest partition first.  Items
// (partitions) are numbered through that order, so the items that leave
// partial results are 0 .. n_records - 1.
struct AttnArgs {
    const uint64_t *k_tab;      // pool tables: K bases then V bases
    const uint8_t *q;           // [L][B][Hq][D]
    const int32_t *tables;      // [B][table_stride]
    float *ws;                  // partial results: [L][n_records][Hq][D + kAttnHeader]
    float *out;                 // [L][B][Hq][D]
    float scale;
    uint32_t num_layers, batch, q_heads, kv_heads, block_size, table_stride;
    uint32_t item_base;         // this launch's first item
    uint32_t layer_items;       // 0: item by item, all layers of one in a row; else layer by
                                // layer, and this many items in this launch
    uint32_t n_records;         // items that leave a partial result
    uint32_t part_tokens;       // most tokens of a partition in this call
    uint32_t item_end[kAttnMaxBatch];  // items of the first s + 1 sequences
    int32_t ctx[kAttnMaxBatch];        // tokens of sequence s
    // its number in the batch (low byte) and its partitions' length in 64
    // tokens (high byte), 16 bits each (in words, for scalar loads)
    uint32_t seq[kAttnMaxBatch / 2];
    // The stage copy a migrating launch carries (read only when it does):
    // logical blocks [mig_from, mig_to) of sequence mig_seq go to the blocks
    // mig_ids[j - mig_from] of the pool whose K and V bases dst_tab lists.
    const uint64_t *dst_tab;
    const int32_t *mig_ids;
    int32_t mig_seq, mig_from, mig_to;
    uint32_t dst_layer_bytes;   // bytes of one destination layer tensor (< 2^31)
    int32_t dst_blocks;         // blocks of the destination pool
};

struct AttnReduceArgs {
    const float *ws;
    float *out;                 // [L][B][Hq][D]
    uint32_t num_layers, batch, q_heads, head_dim, n_records;
    uint64_t row_base;                  // this launch's first row
    uint32_t seqs;                      // sequences of several partitions
    uint32_t seq_end[kAttnMaxBatch];    // records of the first s + 1 of them
    uint8_t seq[kAttnMaxBatch];         // their numbers in the batch
};

// Tokens per partition of a sequence of n tokens cut into `parts` partitions:
// equal shares, whole rounds of the four wavefronts' 16-token groups.
inline int32_t attn_part_len(int32_t n, uint32_t parts)
{
    const uint32_t share = (static_cast<uint32_t>(n) + parts - 1) / parts;
    return static_cast<int32_t>((share + 63) / 64 * 64);
}

// Merges the partitions of each sequence and normalises.  A workgroup takes
// one (layer, sequence, query head) row: its lanes are SUB groups of
// head_dim / 4, each merging every SUB-th partition, eight partitions' loads
// in flight (a record's m and l as one 8-byte load, four sums per lane as one
// 16-byte load); the groups meet in LDS.  SUB = 1 packs several rows into a
// workgroup, for calls of at most eight partitions a sequence.
template <int D, int SUB>
__global__ void __launch_bounds__(kThreads) attn_reduce(const AttnReduceArgs a)
{
    constexpr uint32_t kQuads = D / 4, kRec = D + kAttnHeader;
    constexpr uint32_t kRows = kThreads / (kQuads * SUB);     // rows per workgroup
    static_assert(SUB == 1 || kRows == 1, "several groups: one row per workgroup");
    const uint64_t rows = static_cast<uint64_t>(a.num_layers) * a.seqs * a.q_heads;
    const uint32_t d4 = threadIdx.x % kQuads, sub = SUB > 1 ? threadIdx.x / kQuads : 0u;
    uint64_t r = a.row_base + static_cast<uint64_t>(blockIdx.x) * kRows + (SUB > 1 ? 0u : threadIdx.x / kQuads);
    const bool in = r < rows;
    if (!in)
        r = rows - 1;
    const uint32_t h = r % a.q_heads;
    const uint32_t s = (r / a.q_heads) % a.seqs;
    const uint32_t layer = static_cast<uint32_t>(r / a.q_heads / a.seqs);
    const uint32_t first = s > 0 ? a.seq_end[s - 1] : 0u;
    const int32_t count = static_cast<int32_t>(a.seq_end[s] - first);
    const uint64_t stride = static_cast<uint64_t>(a.q_heads) * kRec;  // one partition
    const float *base = a.ws + ((static_cast<uint64_t>(layer) * a.n_records + first) * a.q_heads + h) * kRec;
    float m = -INFINITY, l = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    auto merge = [&](float m2, float l2, float4 v) {
        const float mm = fmaxf(m, m2);
        if (mm == -INFINITY) {      // no weight on either side; a NaN sum stays one
            l += l2;
            return;
        }
        const float c1 = __expf(m - mm), c2 = __expf(m2 - mm);
        l = l * c1 + l2 * c2;
        acc.x = acc.x * c1 + v.x * c2;
        acc.y = acc.y * c1 + v.y * c2;
        acc.z = acc.z * c1 + v.z * c2;
        acc.w = acc.w * c1 + v.w * c2;
        m = mm;
    };
    for (int32_t p0 = static_cast<int32_t>(sub); p0 < count; p0 += 8 * SUB) {
        float2 ml[8];
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            ml[u] = make_float2(-INFINITY, 0.f);
            v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (p0 + u * SUB < count) {
                const float *src = base + (p0 + u * SUB) * stride;
                ml[u] = *reinterpret_cast<const float2 *>(src);
                v[u] = *reinterpret_cast<const float4 *>(src + kAttnHeader + 4 * d4);
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            merge(ml[u].x, ml[u].y, v[u]);
    }
    if constexpr (SUB > 1) {
        __shared__ float sm[SUB], sl[SUB];
        __shared__ float4 sv[SUB][kQuads];
        sv[sub][d4] = acc;
        if (d4 == 0) {
            sm[sub] = m;
            sl[sub] = l;
        }
        __syncthreads();
        if (sub > 0)
            return;
#pragma unroll
        for (int u = 1; u < SUB; ++u)
            merge(sm[u], sl[u], sv[u][d4]);
    }
    if (in)
        reinterpret_cast<float4 *>(a.out)[((static_cast<uint64_t>(layer) * a.batch + a.seq[s]) * a.q_heads + h) * kQuads +
                                          d4] =
            l > 0.f ? make_float4(acc.x / l, acc.y / l, acc.z / l, acc.w / l) : make_float4(0.f, 0.f, 0.f, 0.f);
}

// ---------------------------------------------------------------------------
// Matrix-core variant.  Per 16-token group of a partition, one wavefront:
//   loads     the group's K and V rows whole, straight from HBM into the
//             wavefront's LDS (global_load_lds_dwordx4: 64 lanes x 16 bytes
//             per instruction, D/8 lanes per row, 256 contiguous bytes a row
//             for D = 128), tokens past the partition's end clamped to its
//             last token (their weights are 0).  The next group's rows are
//             requested as soon as this group's operands have been read out
//             of LDS, so they are in flight while this group computes, and
//             no registers hold rows in transit;
//   S^T = K . Q^T     16 tokens x 16 query rows (the group's heads, then its
//                     last head again, whose results go nowhere),
//                     16x16x32 MFMA over head_dim in steps of 32; the K rows
//                     sit in LDS with their 16-byte chunks XOR-swizzled by
//                     token, so the operand reads (token = lane % 16) hit
//                     distinct banks;
//   online softmax per query row (a lane's rows of S^T are the tokens
//                     4*(lane/16) .. +3 of query row lane%16);
//   O^T += V^T . P^T  16x16x32 MFMA per 16 dims; P^T is already in the
//                     B-operand layout, and V^T comes out of the row-major V
//                     rows through gfx950's transposing LDS read
//                     (ds_read_b64_tr_b16).  P is split into a 16-bit high
//                     part and the 16-bit rounding of the remainder, which
//                     take the two halves of the contraction, so the weights
//                     keep ~2^-16 (bf16) / 2^-22 (fp16) precision.
// The four wavefronts take alternate token groups of the partition and merge
// their states through LDS at the end.  The kernel waits on HBM, not on the
// matrix cores or LDS, so it is built for at least four wavefronts per SIMD (at
// most 128 registers: the accumulators move from AGPRs to VGPRs; 33.5 KiB of
// LDS per workgroup for the rows and the merge, 17.5 for head_dim 64).  The
// carrying variant asks for three only: it also holds the stage's rows between
// LDS and their stores (163 registers for head_dim 128), and at four the
// compiler spills 40 to 52 of them, whose loads and stores the counted wait of
// the loop does not expect.
// What a workgroup spends besides its loop is what bounds short sequences:
// each dependent access costs the latency of a loaded memory system (~5 us
// with every CU's 128 KiB in flight).  So the block ids are one load per lane
// (UNITS), partitions run longest first over all layers (the launch ends on
// short ones), a sequence of one partition needs no record and no merge, and
// results leave in whole rows at device scope.  Measured on MI355X against
// partitions in batch order, layer by layer, ids staged behind a barrier,
// every result through a record and the merge, scattered 64-byte stores
// (lengths evenly spread): 32 layers of 32 heads, 8 sequences of 200-1500
// tokens, 729 -> 522 us (4.90 -> 6.84 TB/s); 64 of 40-300, 962 -> 894; 80 layers
// of 8 heads (64 query heads), 16 of 550-4096, 2048 -> 1926 (6.36 TB/s); 17 of
// 520-3840, 2214 -> 1925; 32 layers of 8 heads, one sequence of 32000, 691 ->
// 671.
// Earlier steps on the same kernel: whole-row K loads rearranged through LDS
// instead of K fragments loaded straight into the operand layout (16 rows x
// 64 bytes per load instruction) +8%; grouping each (partition, layer)'s KV
// heads on one XCD +7%; 2048-token partitions instead of 1024 +4%; rows
// loaded straight into LDS one group ahead instead of through registers, with
// the transposing V^T reads, +2%.
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int BF16>
__device__ __forceinline__ f32x4_t mfma_qk(u32x4 a, u32x4 b, f32x4_t c)
{
    if constexpr (BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                        __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a),
                                                       __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

// The high and the low part of the weights in one 16x16x32 product: k slots
// 8*g4 .. +3 hold the weights' high parts of tokens 4*g4 .. +3, slots + 4 .. 7
// their low parts, against the same V rows twice.
template <int BF16>
__device__ __forceinline__ f32x4_t mfma_pv(uint64_t v, uint64_t hi, uint64_t lo, f32x4_t c)
{
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    return mfma_qk<BF16>(__builtin_bit_cast(u32x4, u64x2{v, v}), __builtin_bit_cast(u32x4, u64x2{hi, lo}), c);
}

// Results leave at device scope (sc1).  On a step whose rows come out of the
// caches (32 layers, 8 KV heads of 8 query heads, 32 sequences of 1000
// tokens) sc1 stores 602 us, nt 612, plain ones 679, no stores at all 533.
constexpr int kResultStore = 16;

// Round a float to the 16-bit type (nearest even); returns the bits.
template <int BF16>
__device__ __forceinline__ uint32_t to16(float x)
{
    if constexpr (BF16) {
        const uint32_t u = __builtin_bit_cast(uint32_t, x);
        return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    } else {
        return __builtin_bit_cast(uint16_t, static_cast<_Float16>(x));
    }
}

__device__ __forceinline__ uint32_t lds_offset(const void *p)
{
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const void LLMIG_LDS *)p));
}

// A group's operands out of LDS: K fragment ks from k_at[ks], V^T fragment mt
// from v_at + 32 * mt.  In assembly, with their wait, because the compiler
// lets every LDS read wait for all outstanding loads into LDS and all stores
// behind them (it cannot tell the group's from the ones still on their way).
template <int KS, int MT>
__device__ __forceinline__ void read_operands(const uint32_t *k_at, uint32_t v_at, u32x4 *kf, uint64_t *vf)
{
    if constexpr (KS == 4) {
        asm volatile("ds_read_b128 %0, %12\n\t"
                     "ds_read_b128 %1, %13\n\t"
                     "ds_read_b128 %2, %14\n\t"
                     "ds_read_b128 %3, %15\n\t"
                     "ds_read_b64_tr_b16 %4, %16\n\t"
                     "ds_read_b64_tr_b16 %5, %16 offset:32\n\t"
                     "ds_read_b64_tr_b16 %6, %16 offset:64\n\t"
                     "ds_read_b64_tr_b16 %7, %16 offset:96\n\t"
                     "ds_read_b64_tr_b16 %8, %16 offset:128\n\t"
                     "ds_read_b64_tr_b16 %9, %16 offset:160\n\t"
                     "ds_read_b64_tr_b16 %10, %16 offset:192\n\t"
                     "ds_read_b64_tr_b16 %11, %16 offset:224\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(kf[0]), "=&v"(kf[1]), "=&v"(kf[2]), "=&v"(kf[3]), "=&v"(vf[0]), "=&v"(vf[1]),
                       "=&v"(vf[2]), "=&v"(vf[3]), "=&v"(vf[4]), "=&v"(vf[5]), "=&v"(vf[6]), "=&v"(vf[7])
                     : "v"(k_at[0]), "v"(k_at[1]), "v"(k_at[2]), "v"(k_at[3]), "v"(v_at)
                     : "memory");
    } else {
        static_assert(KS == 2 && MT == 4, "head_dim 64 or 128");
        asm volatile("ds_read_b128 %0, %6\n\t"
                     "ds_read_b128 %1, %7\n\t"
                     "ds_read_b64_tr_b16 %2, %8\n\t"
                     "ds_read_b64_tr_b16 %3, %8 offset:32\n\t"
                     "ds_read_b64_tr_b16 %4, %8 offset:64\n\t"
                     "ds_read_b64_tr_b16 %5, %8 offset:96\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(kf[0]), "=&v"(kf[1]), "=&v"(vf[0]), "=&v"(vf[1]), "=&v"(vf[2]), "=&v"(vf[3])
                     : "v"(k_at[0]), "v"(k_at[1]), "v"(v_at)
                     : "memory");
    }
}

// Two KiB of K rows and two of V rows as the lanes loaded them.
__device__ __forceinline__ void read_row_pair(uint32_t k_at, uint32_t v_at, u32x4 *k, u32x4 *v)
{
    asm volatile("ds_read_b128 %0, %4\n\t"
                 "ds_read_b128 %1, %4 offset:1024\n\t"
                 "ds_read_b128 %2, %5\n\t"
                 "ds_read_b128 %3, %5 offset:1024\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(k[0]), "=&v"(k[1]), "=&v"(v[0]), "=&v"(v[1])
                 : "v"(k_at), "v"(v_at)
                 : "memory");
}

// Block ids a partition can touch, for the dynamic LDS of attn_partial_mfma
// (UNITS 0): a partition may start inside a block, so at most
// ceil(part_tokens / block_size) + 1 blocks.  A migrating launch keeps the
// destination id of each of them beside it.
__host__ __device__ inline uint32_t attn_blk_slots(uint32_t part_tokens, uint32_t block_size)
{
    return (part_tokens + block_size - 1) / block_size + 1;
}

// MIG: the launch also carries a migration stage of one sequence (Llumnix
// §4.2 stage copy, done as a side effect of decode's reads).  Every
// wavefront already brings its token group's K and V rows (one KV head's
// D * 2 bytes of each token) into LDS; for the tokens of the stage's blocks
// it reads them back out of LDS and stores them, unchanged, at the same
// place in the destination blocks.  Across the kv_heads workgroups of every
// (layer, partition) that covers each whole tile, K and V, of those blocks,
// so the destination receives exactly the bytes a pool-to-pool stage copy
// would write, while HBM reads them once, for the attention (of the
// sequence's partly filled last block, which only a final stage includes,
// the rows of its tokens: the slots past them hold no token).
//
// UNITS: block_size is a multiple of 8, so every 8-token unit of a group
// (partitions start on multiples of 64 tokens) lies in one block: lane l of a
// wavefront looks up the row of its l-th unit once, and a request takes the
// rows of a unit from one lane (v_readlane: a scalar base plus lane offsets
// that never change).  A partition has at most 64 units per wavefront.  Other
// block sizes stage the block ids in LDS and look each token's up.
template <int BF16, int D, int MIG, int UNITS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(MIG ? 3 : 4, 8)))
attn_partial_mfma(const AttnArgs a)
{
    constexpr int KS = D / 32;            // k-steps of the QK product
    constexpr int MT = D / 16;            // 16-dim tiles of the PV product
    constexpr int LPR = D / 8;            // lanes per row in the K and V loads (16 bytes each)
    constexpr int RPL = 64 / LPR;         // rows per load instruction
    constexpr int RB = D * 2;             // bytes of one K or V row
    constexpr int RPB = 128 / D;          // rows per 256 bytes (one pass over the 64 banks)
    constexpr int IPU = KS / 2;           // load instructions per 8-token unit (K and V each)
    constexpr float kLog2e = 1.4426950408889634f;
    // 4 wavefronts x (16 K rows + 16 V rows) in the loop; reused for the
    // final merge of 4 x 16 rows of kMergeRow floats (four of padding).
    constexpr int kMergeRow = D + 4;
    constexpr int kRowBytes = 4 * 2 * 16 * RB, kMergeBytes = 4 * 16 * kMergeRow * 4;
    static_assert(KS * 64 * 16 == 16 * RB, "KS load instructions of 1 KiB cover the 16 rows of a group");
    static_assert(IPU * RPL == 8, "IPU load instructions cover the 8 rows of a unit");
    static_assert(kPartTokens <= 64 * 4 * 8, "a lane per unit of a wavefront's share of a partition");
    __shared__ __align__(16) uint8_t smem[kRowBytes > kMergeBytes ? kRowBytes : kMergeBytes];
    __shared__ float sh_m[4][16], sh_l[4][16];
    // UNITS 0: block ids of the partition, dynamic LDS of attn_blk_slots
    // entries (a migrating launch: twice that, the destination ids after them)
    extern __shared__ int32_t sh_blk[];

    // The dispatcher deals workgroups to the eight XCDs in turn.  Renumbered
    // here so that the kv_heads workgroups of one (item, layer), which read
    // adjacent 256-byte pieces of the same token rows, run one after another
    // on one XCD: linear workgroup w is the (w / 8)-th on XCD w % 8.  The
    // tail of the grid that does not fill whole rounds of 8 * kv_heads keeps
    // the plain order.  Items run longest first, all layers of one after the
    // other, so the last workgroups to run are short ones (see
    // attn_layer_by_layer for the calls that don't).
    uint32_t item, g, layer;
    {
        const uint32_t H = a.kv_heads, lin = blockIdx.x;
        const uint32_t full = gridDim.x - gridDim.x % (8u * H);
        uint32_t unit;                    // (item, layer) in the launch's order
        if (lin < full) {
            const uint32_t k = lin / 8u;
            g = k % H;
            unit = (k / H) * 8u + lin % 8u;
        } else {
            g = lin % H;
            unit = lin / H;
        }
        if (a.layer_items) {
            layer = unit / a.layer_items;
            // (starting one item later in each layer: the items of a layer go to
            // the XCDs in turn, and an even batch would give the longest of every
            // layer to the same one)
            item = (unit - layer * a.layer_items + layer) % a.layer_items;
        } else {
            item = unit / a.num_layers;
            layer = unit - item * a.num_layers;
        }
        item = uniform(item + a.item_base);
        layer = uniform(layer);
    }
    // the item's sequence: the first one whose items end past it
    uint32_t s_lo = 0, s_hi = a.batch - 1;
    while (s_lo < s_hi) {
        const uint32_t mid = (s_lo + s_hi) / 2u;
        if (a.item_end[mid] <= item)
            s_lo = mid + 1u;
        else
            s_hi = mid;
    }
    const uint32_t item_first = s_lo > 0 ? a.item_end[s_lo - 1] : 0u;
    const uint32_t parts = a.item_end[s_lo] - item_first;
    const uint32_t seq = a.seq[s_lo / 2u] >> (16u * (s_lo % 2u));
    const uint32_t b = seq & 0xffu;
    const int32_t ctx = a.ctx[s_lo], plen = static_cast<int32_t>(seq >> 8 & 0xffu) * 64;
    const int32_t start = static_cast<int32_t>(item - item_first) * plen;
    const int32_t end = parts > 1 ? min(ctx, start + plen) : ctx;
    const uint32_t G = a.q_heads / a.kv_heads;
    const uint32_t wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const uint32_t wv = uniform(wave);
    const uint32_t r16 = lane % 16, g4 = lane / 16;
    const int32_t bs = static_cast<int32_t>(a.block_size);

    const uint8_t *kbase = reinterpret_cast<const uint8_t *>(table_entry(a.k_tab, layer));
    const uint8_t *vbase = reinterpret_cast<const uint8_t *>(table_entry(a.k_tab, a.num_layers + layer));

    // A migrating launch: whether this workgroup's rows are the migrating
    // sequence's.
    const bool mig = MIG && static_cast<int32_t>(b) == a.mig_seq;
    const int32_t *table = a.tables + static_cast<uint64_t>(b) * a.table_stride;
    const int32_t tg0 = start + 16 * static_cast<int32_t>(wv);
    const int32_t first_blk = UNITS ? 0 : start / bs;
    int32_t *sh_dst = sh_blk + attn_blk_slots(a.part_tokens, a.block_size);
    // UNITS: lane l's unit is tokens tg0 + 64 * (l / 2) + 8 * (l % 2) .. + 7:
    // the slot (block * block_size + slot in it) of its first token, or, past
    // the partition's end, of the partition's last token; and where the unit
    // lands in the destination pool (-1: not in the stage).
    uint32_t unit_slot = 0;
    int32_t unit_dst = -1;
    if constexpr (UNITS) {
        if (tg0 < end) {
            const int32_t t = min(tg0 + 64 * static_cast<int32_t>(lane / 2) + 8 * static_cast<int32_t>(lane % 2), end - 1);
            const int32_t blk = t / bs;
            unit_slot = static_cast<uint32_t>(table[blk]) * a.block_size + static_cast<uint32_t>(t - blk * bs);
            if (mig && blk >= a.mig_from && blk < a.mig_to) {
                const int32_t id = a.mig_ids[blk - a.mig_from];
                if (id >= 0 && id < a.dst_blocks)      // an id outside the pool is not written
                    unit_dst = id * bs + (t - blk * bs);
            }
        }
    } else {
        // the partition's block ids, once, and the destination block of each
        // of its logical blocks (-1 outside the stage)
        const int32_t n_blk = end > start ? (end - 1) / bs - first_blk + 1 : 0;
        for (int32_t k = threadIdx.x; k < n_blk; k += kThreads)
            sh_blk[k] = table[first_blk + k];
        if (mig) {
            for (int32_t k = threadIdx.x; k < n_blk; k += kThreads) {
                const int32_t j = first_blk + k;
                const int32_t id = j >= a.mig_from && j < a.mig_to ? a.mig_ids[j - a.mig_from] : -1;
                sh_dst[k] = id < a.dst_blocks ? id : -1;     // an id past the pool is not written
            }
        }
        __syncthreads();
    }

    // Q^T fragments (B operand): query row r16 of the group, dims 32*ks + 8*g4
    // .. +8; rows past the group: the last one again, whose results go nowhere.
    u32x4 qf[KS];
    const uint64_t q_row = (static_cast<uint64_t>(layer) * a.batch + b) * a.q_heads + g * G + min(r16, G - 1u);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        qf[ks] = load16(a.q + (q_row * D + 32 * ks + 8 * g4) * 2);
    const float qk_scale = a.scale * kLog2e;
    float m = -INFINITY, lsum = 0.f;
    f32x4_t acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
        acc[mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // The wavefront's rows of one 16-token group in LDS, D/8 chunks of 16
    // bytes a row.  K chunk c of local token t sits at slot c ^ kswz(t), so
    // that the 16 tokens an operand read touches at once fall on distinct
    // banks; V rows are plain (the transposing reads take them as they are).
    uint8_t *kbuf = smem + wv * (2 * 16 * RB);
    uint8_t *vbuf = kbuf + 16 * RB;
    auto kswz = [](uint32_t t) { return (t / RPB) % LPR; };
    // Requests the rows of the group starting at token t0: KS instructions
    // for K and KS for V, instruction j's lane carrying local token
    // j*RPL + lane/LPR into LDS slot lane%LPR of that token's row.  A token
    // past the partition's end loads its last token; its score is masked
    // below, so its weight is 0.
    const uint32_t lrow = lane / LPR, lslot = lane % LPR;
    const uint32_t row_bytes = a.kv_heads * RB;             // one token's rows of every KV head
    auto load_rows = [&](int j, const uint8_t *k, const uint8_t *v) {
        __builtin_amdgcn_global_load_lds((const void LLMIG_GLOBAL *)k, (void LLMIG_LDS *)(kbuf + j * 1024), 16, 0,
                                         kStreamLoad);
        __builtin_amdgcn_global_load_lds((const void LLMIG_GLOBAL *)v, (void LLMIG_LDS *)(vbuf + j * 1024), 16, 0,
                                         kStreamLoad);
    };
    auto request_group = [&](int32_t t0) {
        if constexpr (UNITS) {
            const uint32_t u0 = static_cast<uint32_t>(t0 - tg0) / 32u;      // the group's first unit (lane)
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const uint32_t slot = __builtin_amdgcn_readlane(unit_slot, u0 + half);
                const uint64_t base = (static_cast<uint64_t>(slot) * a.kv_heads + g) * RB;
                // rows of the unit that hold tokens of the partition, less one
                const int32_t last = max(min(end - 1 - (t0 + 8 * half), 7), 0);
#pragma unroll
                for (int i = 0; i < IPU; ++i) {
                    const int j = half * IPU + i;
                    const uint32_t row = min(static_cast<uint32_t>(i * RPL) + lrow, static_cast<uint32_t>(last));
                    const uint32_t off = row * row_bytes;
                    load_rows(j, kbase + base + off + 16 * (lslot ^ kswz(j * RPL + lrow)),
                              vbase + base + off + 16 * lslot);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                const uint32_t tl = j * RPL + lrow;
                const int32_t t = min(t0 + static_cast<int32_t>(tl), end - 1);
                const uint64_t row = (static_cast<uint64_t>(sh_blk[t / bs - first_blk]) * a.block_size + t % bs) *
                                         a.kv_heads + g;
                load_rows(j, kbase + (row * D + 8 * (lslot ^ kswz(tl))) * 2, vbase + (row * D + 8 * lslot) * 2);
            }
        }
    };
    // A migrating launch: stores the group's rows that belong to the stage's
    // blocks into the destination pool.  Lane `lane` of load instruction j
    // brought token j*RPL + lane/LPR's chunk lane%LPR of the row (K: the
    // swizzled slot of the chunk) into LDS at j * 1024 + lane * 16; it reads
    // that back and stores it where the chunk lives in the destination tile:
    // (slot of the token, head g, the chunk).  Rows of tokens past the
    // partition's end (loaded as copies of its last token) are skipped.
    // Split in two, so that the next group's request goes out in between.
    u32x4 rows_k[KS], rows_v[KS];
    auto read_rows = [&]() {
#pragma unroll
        for (int j = 0; j < KS; j += 2)
            read_row_pair(lds_offset(kbuf) + j * 1024 + lane * 16, lds_offset(vbuf) + j * 1024 + lane * 16, rows_k + j,
                          rows_v + j);
    };
    auto store_rows = [&](int32_t tg) {
        // raw buffer stores over the destination layer tensors, with the
        // migration copy's cache policy (streaming, device scope); a whole
        // 10.7 GB stage carried by one GQA decode step added 2.2-2.8 ms to
        // the step with them, 2.8-2.9 ms with plain non-temporal stores.
        // A row that is not the stage's gets an offset past the resource
        // (layer tensors are under 2^31 bytes), so the range check drops
        // its store and every store runs unpredicated.
        constexpr uint32_t kDropped = 0x80000000u;
        const __amdgpu_buffer_rsrc_t rk = tile_rsrc(
            reinterpret_cast<const uint8_t *>(table_entry(a.dst_tab, layer)), a.dst_layer_bytes);
        const __amdgpu_buffer_rsrc_t rv = tile_rsrc(
            reinterpret_cast<const uint8_t *>(table_entry(a.dst_tab, a.num_layers + layer)), a.dst_layer_bytes);
        uint32_t off[KS];
        if constexpr (UNITS) {
            const uint32_t u0 = static_cast<uint32_t>(tg - tg0) / 32u;
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                const int32_t d = static_cast<int32_t>(__builtin_amdgcn_readlane(unit_dst, u0 + j / IPU));
                const uint32_t row = (j % IPU) * RPL + lrow;
                off[j] = d < 0 || tg + j * RPL + static_cast<int32_t>(lrow) >= end
                             ? kDropped
                             : (static_cast<uint32_t>(d) * a.kv_heads + g) * RB + row * row_bytes;
            }
        } else {
            const uint32_t tile = a.block_size * row_bytes;
            const int32_t q = tg / bs, r0 = tg - q * bs;          // the group's first token: block, slot
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                const int32_t tl = j * RPL + static_cast<int32_t>(lrow);
                const int32_t s = r0 + tl, bo = s / bs, slot = s - bo * bs;
                const int32_t d = tg + tl < end ? sh_dst[q + bo - first_blk] : -1;
                off[j] = d < 0 ? kDropped
                               : static_cast<uint32_t>(d) * tile + (static_cast<uint32_t>(slot) * a.kv_heads + g) * RB;
            }
        }
#pragma unroll
        for (int j = 0; j < KS; ++j)
            buffer_store16(rk, off[j] + 16 * ((lane % LPR) ^ kswz(j * RPL + lane / LPR)), rows_k[j]);
#pragma unroll
        for (int j = 0; j < KS; ++j)
            buffer_store16(rv, off[j] + 16 * (lane % LPR), rows_v[j]);
    };
    // whether the group starting at token tg holds tokens of the stage's
    // blocks (wavefront-uniform)
    auto carries = [&](int32_t tg) {
        return MIG && mig && (tg + 15) / bs >= a.mig_from && tg / bs < a.mig_to;
    };
    if (tg0 < end)
        request_group(tg0);
    // K fragments (A operand): token r16, dims 32*ks + 8*g4 .. +8.  V^T
    // fragments (A operand of O^T: dim 16*mt + r16, tokens 4*g4 .. +3) by
    // transposing reads: lane r16 of the 16-lane group g4 receives element
    // r16 % 4 of the 8 bytes that lane 4*q + r16/4 of its group addresses, for
    // q = 0..3; those address token 4*g4 + q, dims 16*mt + 4*(r16 % 4) .. +3.
    uint32_t k_at[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        k_at[ks] = lds_offset(kbuf) + r16 * RB + ((4 * ks + g4) ^ kswz(r16)) * 16;
    const uint32_t v_at = lds_offset(vbuf) + (4 * g4 + r16 / 4) * RB + 4 * (r16 % 4) * 2;
    // The query rows have landed too; said here, so that the compiler puts no
    // wait for them, and with it for every store, into the loop.
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        asm volatile("" : "+v"(qf[ks]));
    bool stored = false;    // the group before this one issued 2 * KS stores, after this one's request
    for (int32_t tg = tg0; tg < end; tg += 64) {
        // this group's rows have landed; loads and stores complete in order,
        // so the stores behind them need not have
        if (MIG && stored)
            __builtin_amdgcn_s_waitcnt(kWaitVm0 | (2 * KS));
        else
            __builtin_amdgcn_s_waitcnt(kWaitVm0);
        u32x4 kf[KS];
        uint64_t vf[MT];
        read_operands<KS, MT>(k_at, v_at, kf, vf);
        const bool carry = carries(tg);
        if (carry)
            read_rows();
        // (the reads have returned: the next group's rows may overwrite them)
        if (tg + 64 < end)
            request_group(tg + 64);
        if (MIG) {
            // the stores stay behind the request: the wait above counts on it
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            if (carry)
                store_rows(tg);
            stored = carry;
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
        // S^T = K . Q^T
        f32x4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            s = mfma_qk<BF16>(kf[ks], qf[ks], s);
        // online softmax for query row r16 over tokens tg + 4*g4 + i
        float sc[4], mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sc[i] = tg + static_cast<int32_t>(4 * g4) + i < end ? s[i] * qk_scale : -INFINITY;
            mx = fmaxf(mx, sc[i]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        // A maximum of -inf (every score so far is) must not be subtracted:
        // where a partition starts decides what "so far" holds.
        const float m_new = fmaxf(m, mx), m_sub = m_new == -INFINITY ? 0.f : m_new;
        const float c = exp2f(m - m_sub);
        float p[4], ps = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = exp2f(sc[i] - m_sub);
            ps += p[i];
        }
        ps += __shfl_xor(ps, 16);
        ps += __shfl_xor(ps, 32);
        lsum = lsum * c + ps;
        m = m_new;
        uint64_t ph = 0, pl = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t hi = to16<BF16>(p[i]);
            const float hv = BF16 ? __builtin_bit_cast(float, hi << 16)
                                  : static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(hi)));
            ph |= static_cast<uint64_t>(hi) << (16 * i);
            pl |= static_cast<uint64_t>(to16<BF16>(p[i] - hv)) << (16 * i);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            acc[mt] = acc[mt] * c;
            acc[mt] = mfma_pv<BF16>(vf[mt], ph, pl, acc[mt]);
        }
    }

    // Merge the four wavefronts (each holds, of query row r16, its maximum,
    // its weight sum and O^T rows 16*mt + 4*g4 + i) through LDS, as rows of
    // kMergeRow floats, so that the results leave in whole rows: a workgroup
    // ends only when its stores are acknowledged, and scattered 64-byte
    // pieces kept it waiting.
    __syncthreads();                                // every wave is done with its rows
    float *so = reinterpret_cast<float *>(smem);    // [wave][query row][kMergeRow]
    if (g4 == 0) {
        sh_m[wave][r16] = m;
        sh_l[wave][r16] = lsum;
    }
    if (r16 < G) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            *reinterpret_cast<f32x4_t *>(so + (wave * 16 + r16) * kMergeRow + 16 * mt + 4 * g4) = acc[mt];
    }
    __syncthreads();
    // the sequence's output if it is one partition, else a record; of the
    // group's query heads
    const bool whole = parts == 1;
    const uint32_t out_row = whole ? D : D + kAttnHeader, out_at = whole ? 0u : kAttnHeader;
    const uint64_t out_first = whole ? static_cast<uint64_t>(layer) * a.batch + b
                                     : static_cast<uint64_t>(layer) * a.n_records + item;
    const __amdgpu_buffer_rsrc_t ro = tile_rsrc(
        reinterpret_cast<const uint8_t *>((whole ? a.out : a.ws) + (out_first * a.q_heads + g * G) * out_row),
        G * out_row * 4);
    auto put = [&](uint32_t at, f32x4_t v) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), ro, at * 4, 0, kResultStore);
    };
    for (uint32_t x = threadIdx.x; x < G * (D / 4); x += kThreads) {
        const uint32_t row = x / (D / 4), d4 = x % (D / 4);
        float mm = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            mm = fmaxf(mm, sh_m[w][row]);
        float ll = 0.f;
        f32x4_t o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float c = mm == -INFINITY ? 0.f : exp2f(sh_m[w][row] - mm);
            ll += sh_l[w][row] * c;
            o += *reinterpret_cast<const f32x4_t *>(so + (w * 16 + row) * kMergeRow + 4 * d4) * c;
        }
        if (whole)                  // as the merge kernel: zeros where there is no finite weight sum
            o = ll > 0.f ? o / ll : f32x4_t{0.f, 0.f, 0.f, 0.f};
        put(row * out_row + out_at + 4 * d4, o);
        // the reduce kernel merges with natural exponentials: m in that base
        if (!whole && d4 == 0)
            put(row * out_row, f32x4_t{mm == -INFINITY ? -INFINITY : mm / kLog2e, ll, 0.f, 0.f});
    }
}

template <int BF16, int D>
const void *attn_kernel(bool migrating, bool units)
{
    if (migrating)
        return units ? reinterpret_cast<const void *>(&attn_partial_mfma<BF16, D, 1, 1>)
                     : reinterpret_cast<const void *>(&attn_partial_mfma<BF16, D, 1, 0>);
    return units ? reinterpret_cast<const void *>(&attn_partial_mfma<BF16, D, 0, 1>)
                 : reinterpret_cast<const void *>(&attn_partial_mfma<BF16, D, 0, 0>);
}

const void *attn_kernel_for(int bf16, int head_dim, int group, bool migrating, bool units)
{
    if (group < 1 || group > 16 || (group & (group - 1)) != 0)
        return nullptr;
    if (head_dim == 64)
        return bf16 ? attn_kernel<1, 64>(migrating, units) : attn_kernel<0, 64>(migrating, units);
    if (head_dim == 128)
        return bf16 ? attn_kernel<1, 128>(migrating, units) : attn_kernel<0, 128>(migrating, units);
    return nullptr;
}

// ---------------------------------------------------------------------------
// How a call is cut into partitions.

// Partitions of a sequence of n tokens, at most `part` tokens each.
inline uint32_t attn_parts(int32_t n, int32_t part)
{
    if (n <= part)
        return 1u;
    const uint32_t parts = (static_cast<uint32_t>(n) + part - 1) / part;
    const uint32_t len = attn_part_len(n, parts);    // rounded up to 64: perhaps fewer are enough
    return (static_cast<uint32_t>(n) + len - 1) / len;
}

// Bytes of the partial results of a call (sequences of one partition leave none).
inline int attn_record_bytes(const int32_t *ctx_lens, int32_t batch, int32_t part, int64_t num_layers,
                             int64_t q_heads, int64_t head_dim, int64_t *bytes)
{
    int64_t n = 0, v = 0;
    for (int32_t b = 0; b < batch; ++b) {
        const uint32_t parts = attn_parts(ctx_lens[b], part);
        n += parts > 1 ? parts : 0;
    }
    if (__builtin_mul_overflow(num_layers, n, &v) || __builtin_mul_overflow(v, q_heads, &v) ||
        __builtin_mul_overflow(v, (head_dim + kAttnHeader) * 4, &v))
        return LLMIG_EINVAL;
    *bytes = v;
    return LLMIG_OK;
}

// Most tokens per partition of a call: kPartTokens, unless that leaves the
// chip short of workgroups.  A partition costs a workgroup's start and end
// (block ids, query rows, the first rows' latency, the merge, a record) and a
// share of the merge kernel, so a call is cut no finer than fills the chip,
// counted in workgroups: one a CU for head_dim 128, two (of half the bytes)
// for 64 and for calls of no sequence over 2048 tokens, whose workgroups are
// short.  Past that a cut can only even out the CUs: calls that need the merge
// anyway are cut to the next whole number a CU, up to three.  Measured, partitions
// of 2048 / 1536 / 1024 / 768 / 512 / 384 / 256 tokens (workgroups), us:
//   head_dim 128, 8 heads, three of up to 9280: 34.5 (88), 31.7, 27.4, 25.3
//     (224), 27.2 (328), 26.1, 27.1; 4 heads, 28 of up to 4170: 37.5 (160),
//     30.2, 29.0 (256), 31.9, 30.1, 31.9, 32.1
//   two a CU: five of up to 29082, 71.0 (336), 67.0 (448), 68.3 (664), 68.4
//   three a CU: 4 layers of 13 heads, seven of up to 6412, 91.3 (624), 84.5
//     (768); 8 layers of 8, four of up to 6823, 90.0 (576), 85.6 (768); four a
//     CU: 640 to 990 workgroups, level
//   head_dim 64, 4 heads, 14 of up to 11364: 29.3 (156), 26.3, 24.2 (268),
//     22.8, 21.7 (508), 22.7, 22.4; 32 heads, 2 of 23635: 50.6 (480), 55.3
//     (640), 54.9, 53.9, 51.8
// The merge is a launch of its own, so a call of short sequences stays whole
// (two of up to 757 13.8 against 15 cut, 16 of up to 569 12.6 and 15.3, two of
// up to 933 17.0 and 13.8), and so does one whose longest partition would
// become less than a quarter shorter (a tenth, where the merge is needed
// anyway).  head_dim 128, one layer, whole / 256 / 512 workgroups: 8 heads, 30
// of up to 2003 41.1 / 35.5 / 28.3, 58 of 4 heads up to 1422 30.4 / 28.2 / 23.9,
// 59 of 8 heads up to 1202 (472) level.
constexpr int64_t kAttnCUs = 256, kAttnWorkgroupsMost = 3 * kAttnCUs;

// Workgroups per layer and KV head of a call cut into partitions of at most
// `part` tokens.
inline int64_t attn_items(const int32_t *ctx_lens, int32_t batch, int32_t part)
{
    int64_t n = 0;
    for (int32_t b = 0; b < batch; ++b)
        n += attn_parts(ctx_lens[b], part);
    return n;
}

inline int32_t attn_part_tokens(const int32_t *ctx_lens, int32_t batch, int64_t num_layers, int64_t kv_heads,
                                int64_t head_dim)
{
    int32_t longest = 0;
    for (int32_t b = 0; b < batch; ++b)
        longest = std::max(longest, ctx_lens[b]);
    int64_t per_item = 0, whole = 0;
    if (longest <= kWholeTokens || __builtin_mul_overflow(num_layers, kv_heads, &per_item) ||
        __builtin_mul_overflow(per_item, attn_items(ctx_lens, batch, kPartTokens), &whole))
        return kPartTokens;
    const bool merges = longest > kPartTokens;
    int64_t most = head_dim == 64 || !merges ? 2 * kAttnCUs : kAttnCUs;
    while (whole > most && most < kAttnWorkgroupsMost && merges)
        most += kAttnCUs;
    if (whole > most)
        return kPartTokens;
    int32_t lo = kMinPartTokens / 64, hi = kPartTokens / 64;    // the shortest that keeps to `most`
    while (lo < hi) {
        const int32_t mid = (lo + hi) / 2;
        if (attn_items(ctx_lens, batch, 64 * mid) * per_item <= most)
            hi = mid;
        else
            lo = mid + 1;
    }
    return 100 * 64 * lo > (merges ? 90 : 75) * std::min(longest, kPartTokens) ? kPartTokens : 64 * lo;
}

// Workgroups a CU that calls of long partitions keep to, by asking for LDS they
// don't use (0: as many as fit): with every slot taken more rows are in flight
// than the memory system needs, and each workgroup's own waits (its start, its
// end) last as long as that queue.  Three for head_dim 128, four (of up to
// eight) for 64.  32 layers, head_dim 64, 32 heads, mean partition 860 / 1350 /
// 2048 tokens 137.9 -> 132.7, 170 -> 161, 233 -> 223 us (600 tokens: level, 140:
// 99 -> 111); head_dim 128, 2000 tokens 658 -> 651, 479 -> 472 (860 tokens: 270 ->
// 272).  Where that leaves a second round of a few workgroups it loses: 8
// layers of 13 heads of 64, two of up to 17421 (1144 workgroups) 98 -> 106,
// 1248 87 -> 92, 1408 110 -> 117; 1504 gain 7%.  Calls just short of 1024
// workgroups run as two rounds of two a CU: one layer of 4 heads of 64, 38 of
// up to 25627 (944) 90 -> 84.5, 8 heads, 28 of up to 14959 (904) 88 -> 75;
// head_dim 128, 64 of up to 6197 (936) 147 -> 136; 800 workgroups lose 6%.  A
// call that carries a stage, whose workgroups differ in length anyway, keeps
// to the first rule alone: 4 layers of 32 heads of 64, one of 16528 (1152
// workgroups) 250 us with four a CU, 267 with eight.
inline int attn_workgroups_per_cu(int64_t head_dim, int64_t workgroups, int64_t mean_tokens, bool migrating)
{
    const int64_t full = head_dim == 64 ? 4 : 3;
    if (!migrating && workgroups >= 840 && workgroups <= 4 * kAttnCUs && mean_tokens >= 1200)
        return 2;
    if (!migrating && 5 * workgroups < 7 * full * kAttnCUs)
        return 0;
    return mean_tokens >= (head_dim == 64 ? 800 : 1500) ? full : 0;
}

// Whether a call runs layer by layer instead of longest item first: batches of
// many short sequences of head_dim 64, whose neighbours then read and write one
// layer's tensors (what exactly that saves was not traced).  Longest first ->
// layer by layer: 80 layers of 8 heads, 38 of up to 120 tokens 89.9 -> 80.4 us,
// 64 of up to 400 354 -> 321, 46 of 25, 29 of up to 125 117 -> 107, 32 of 32, 24
// of up to 400 154 -> 144 (176 with the layers' items in one order on the XCDs, 8
// of up to 400 72 -> 106), 8 of up to 40 level.
// Elsewhere the end of the launch decides: 73 layers of 4 heads of 64, 32 of up
// to 633 (mean 280) 14% slower, 80 of 8 heads of 128, 12 of up to 122 (7680
// workgroups) 51 -> 55, decode steps of long sequences up to 48% slower.  A launch
// that carries a stage keeps to longest first: 32 layers of 32 heads, 40 of up to
// 400 tokens 366 -> 415 us, 60 of 13, 62 of up to 417 396 -> 428.
inline bool attn_layer_by_layer(int64_t head_dim, int64_t workgroups, int64_t mean_tokens)
{
    return head_dim == 64 && workgroups >= 8192 && mean_tokens < 200;
}

// Whether the sequence whose stage a call carries is launched apart, before the
// others, which then run in the kernel that carries none: many short sequences.
// A carrying workgroup holds the stage's rows in registers (163 against 120 for
// head_dim 128, 96 against 74 for 64), so fewer of them share a CU, and of short
// sequences, all start and end, it is the number in flight that counts.  One
// launch -> two: 51 layers of 34 heads of 128, 15 of up to 75 tokens 164 -> 143
// us; 80 of 8, 30 of up to 150 162 -> 153; 28 of 32 heads of 64, 53 of up to 100
// 166 -> 154; 80 of 8, 25 of up to 120 (16000 workgroups) 70 -> 66.  The second
// launch costs the end of the first: 80 layers of 8 heads of 128, 12 of up to 240
// (7680 workgroups) 104 -> 107, 50 of 8, 41 of up to 418 (mean 180) 293 -> 296, 64
// of up to 1000 1671 -> 1687.
inline bool attn_carry_apart(int64_t workgroups, int64_t mean_tokens)
{
    return workgroups >= 16000 && mean_tokens < 160;
}

// Dynamic LDS that keeps n workgroups of the partial kernel a CU (160 KiB of
// LDS; 17.5 KiB a workgroup for head_dim 64, 33.5 for 128).
inline size_t attn_spare_lds(int64_t head_dim, int n)
{
    return n == 0 ? 0 : n == 2 ? (head_dim == 64 ? 40000 : 24000) : 15000;
}

// The merge kernel for at most `most` partitions a sequence; returns its rows
// per workgroup.
inline uint32_t attn_reduce_kernel(int head_dim, uint32_t most, const void **fn)
{
    if (head_dim == 64) {
        *fn = most <= 8 ? reinterpret_cast<const void *>(&attn_reduce<64, 1>)
                        : reinterpret_cast<const void *>(&attn_reduce<64, 16>);
        return most <= 8 ? kThreads / 16 : 1;
    }
    *fn = most <= 8 ? reinterpret_cast<const void *>(&attn_reduce<128, 1>)
                    : reinterpret_cast<const void *>(&attn_reduce<128, 8>);
    return most <= 8 ? kThreads / 32 : 1;
}

} // namespace

"""The uncapped tile copy (one 1 KiB row per wavefront) where its dispatch
turns, byte for byte against the CPU oracle: launches on both sides of the
small-launch rule, on both sides of the rule that hands each XCD runs of rows
(whole rounds, a ragged tail, less than one round), pairs in the caller's
order and pairs ordered by destination, 16-bit, 32-bit and device ids, several
launches, tiles that are not whole rows, and staging buffers on either side
(where reordered pairs carry their place in the buffer)."""
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import HostPool
from paper_2406_03243_amd import harness
from paper_2406_03243_amd import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2406_03243_amd import llmig
    from paper_2406_03243_amd.llmig import Pool

# layers, blocks, block_size, heads, head_dim, pairs
CASES = [
    (1, 40, 16, 32, 128, 31),       # 7936 rows: the small launch; under one round of runs
    (1, 40, 16, 32, 128, 32),       # 8192 rows: the last small launch
    (1, 40, 16, 32, 128, 33),       # 8448 rows: two whole rounds and a tail
    (2, 200, 16, 33, 128, 61),      # 132 KiB tiles: runs that cross tiles, a ragged tail
    (1, 80, 16, 31, 128, 70),       # 124 KiB tiles: rows dealt in turn
    (3, 700, 16, 3, 64, 600),       # 6 KiB tiles, 512 + 88 pairs
    (2, 1500, 8, 5, 40, 1100),      # 3200-byte tiles: a partial last row, three launches
    (1, 66000, 1, 1, 24, 9000),     # 48-byte tiles, ids past 16 bits
    (1, 220, 16, 32, 128, 200),     # 50 MiB: ordered by destination
    (2, 2500, 16, 4, 128, 1000),    # ordered, ids past 11 bits, several launches
]


def image(pool) -> HostPool:
    return HostPool(harness.snapshot(pool.k), harness.snapshot(pool.v), pool.block_size, pool.slot_bytes)


def pool(shape, seed, purpose):
    k, v = harness.alloc_layers(shape)
    total = sum(t.numel() * t.element_size() for t in k + v)
    harness.fill_bytes_from_host(k + v, wl.random_bytes(seed, purpose, total))
    return Pool(k, v)


def where(ids, dev):
    return torch.from_numpy(ids).cuda() if dev else ids


@pytest.mark.parametrize("dev", [False, True], ids=["host", "device"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"T{c[2] * c[3] * c[4] * 2}_n{c[5]}")
def test_copy_rows(case, dev):
    print("[case]", case, dev, flush=True)
    sys.stdout.flush()
    layers, blocks, bs, heads, dim, n = case
    shape = wl.PoolShape(layers, blocks, bs, heads, dim, "fp16")
    src, dst = pool(shape, 60 + n, wl.SRC_VALUES), pool(shape, 60 + n, wl.DST_VALUES)
    g = wl.stream(60 + n, wl.EXTRA)
    ms, md = (g.choice(blocks, n, replace=False).astype(np.int32) for _ in range(2))
    hs, hd = image(src), image(dst)
    orc = oracle.default()
    llmig.llmig_stage(src, dst, where(ms, dev), where(md, dev))
    torch.cuda.synchronize()
    orc.copy(hs, hd, ms, md)
    assert image(dst).equals(hd) and image(src).equals(hs), "stage differs from the oracle"
    # the same blocks through staging; a gather may repeat a block
    rep = ms.copy()
    rep[n // 2] = rep[0]
    staging = torch.full((n * layers * 2 * src.tile_bytes + 64,), 7, dtype=torch.uint8, device="cuda")
    llmig.llmig_pack(src, where(rep, dev), staging[:-64])
    torch.cuda.synchronize()
    want = orc.pack(hs, rep)
    assert np.array_equal(staging[:-64].cpu().numpy(), want) and bool((staging[-64:] == 7).all()), "pack differs"
    into = g.choice(blocks, n, replace=False).astype(np.int32)
    llmig.llmig_unpack(dst, where(into, dev), staging[:-64])
    torch.cuda.synchronize()
    orc.unpack(hd, into, want)
    assert image(dst).equals(hd), "unpack differs"


# converting stages of more than one round of XCD runs, slabs of 1 to 16
# wavefronts: layers, blocks, block_size, heads, head_dim, pairs
CONVERT_CASES = [
    (1, 60, 8, 3, 64, 50),          # 1 KiB slabs
    (2, 80, 16, 5, 40, 70),         # 80 chunks: a partial second wavefront
    (1, 40, 16, 13, 128, 33),       # 858 slabs: one round of runs and a tail
    (1, 40, 32, 9, 128, 31),        # 8 KiB slabs
    (1, 34, 64, 2, 128, 34),        # 16 KiB slabs
    (1, 600, 8, 2, 16, 530),        # 256-byte slabs, two launches
    (1, 1000, 16, 16, 128, 500),    # ordered by destination
]


@pytest.mark.parametrize("dev", [False, True], ids=["host", "device"])
@pytest.mark.parametrize("case", CONVERT_CASES, ids=lambda c: f"slab{c[2] * c[4] * 2}_n{c[5]}")
def test_convert_slabs(case, dev):
    print("[case]", case, dev, flush=True)
    layers, blocks, bs, heads, dim, n = case
    shape = wl.PoolShape(layers, blocks, bs, heads, dim, "fp16")
    orc = oracle.default()
    for sl, dl in (((0, 0), (1, 1)), ((0, 1), (2, 3)), ((2, 3), (0, 0)), ((3, 2), (1, 1)), ((1, 0), (1, 3))):
        src, dst = pool(shape, 80 + n, wl.SRC_VALUES), pool(shape, 80 + n, wl.DST_VALUES)
        src = Pool(src.k, src.v, sl)
        dst = Pool(dst.k, dst.v, dl)
        g = wl.stream(80 + n, wl.EXTRA)
        ms, md, into = (g.choice(blocks, n, replace=False).astype(np.int32) for _ in range(3))
        hs, hd = image(src), image(dst)
        llmig.llmig_stage(src, dst, where(ms, dev), where(md, dev))
        torch.cuda.synchronize()
        orc.copy_layout(hs, sl, hd, dl, ms, md, heads, dim, 2)
        assert image(dst).equals(hd) and image(src).equals(hs), f"stage {sl} -> {dl} differs from the oracle"
        packed = orc.pack(hs, ms)
        llmig.llmig_unpack_layout(dst, where(into, dev), torch.from_numpy(packed).cuda(), sl)
        torch.cuda.synchronize()
        orc.unpack_layout(hd, dl, into, packed, sl, heads, dim, 2)
        assert image(dst).equals(hd), f"converting unpack {sl} -> {dl} differs"


# layers, blocks, block_size, heads, head_dim, first token, tokens
WRITE_CASES = [
    (2, 12, 16, 3, 64, 5, 1),        # one token: no slab
    (2, 12, 16, 3, 64, 15, 2),       # the last slot of a block and the first of the next
    (1, 12, 16, 13, 128, 0, 32),     # whole blocks
    (2, 12, 16, 5, 40, 3, 70),       # partial first and last blocks, 80-chunk slabs
    (1, 300, 8, 2, 64, 4, 2100),     # 8-token units, more blocks than one launch carries
    (1, 20, 32, 3, 128, 9, 200),     # partial 8-token units on both ends
    (1, 20, 12, 3, 64, 7, 100),      # HDN with a block size that 8 does not divide
    (1, 6, 128, 2, 128, 100, 400),   # slabs over 16 KiB
    (1, 140, 16, 32, 128, 5, 2060),  # a prompt of 8 KiB slots
    (2, 12, 16, 8, 128, 9, 64),      # the longest append of 2 KiB slots
    (2, 12, 16, 8, 128, 9, 65),      # the shortest prompt
]


@pytest.mark.parametrize("layouts", [(0, 0), (1, 1), (2, 3), (3, 2), (0, 3)], ids=lambda l: f"{l[0]}{l[1]}")
@pytest.mark.parametrize("case", WRITE_CASES, ids=lambda c: f"bs{c[2]}_at{c[5]}_n{c[6]}")
def test_write_tokens(case, layouts):
    print("[case]", case, layouts, flush=True)
    layers, blocks, bs, heads, dim, first, n = case
    base = pool(wl.PoolShape(layers, blocks, bs, heads, dim, "bf16"), 90 + n, wl.DST_VALUES)
    dst = Pool(base.k, base.v, layouts)
    table = wl.stream(90 + n, wl.EXTRA).permutation(blocks).astype(np.int32)
    data = wl.random_bytes(90 + n, wl.APPEND_VALUES, layers * 2 * n * heads * dim * 2).reshape(
        layers, 2, n, heads * dim * 2)
    hd = image(dst)
    llmig.llmig_write_tokens(dst, table, first, torch.from_numpy(data).cuda())
    torch.cuda.synchronize()
    oracle.default().write_tokens_layout(hd, layouts, table, first, data, heads, dim, 2)
    assert image(dst).equals(hd), "differs from the oracle"

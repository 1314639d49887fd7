"""What the library's calls launch (CPU only): the built library over a
stand-in HIP runtime that records launches instead of running them, in a
process of its own (launch_recorder.py).  Each rule is checked on both of its
sides, and that the launches of a call cover its work exactly once."""
import json
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

import attn_cases
from paper_2406_03243_amd.build import LIBRARY

TESTS = os.path.dirname(os.path.abspath(__file__))
pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc missing")


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    fake = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", fake, os.path.join(TESTS, "fake_hip.c")], check=True)

    def run(calls):
        res = subprocess.run([sys.executable, os.path.join(TESTS, "launch_recorder.py"), fake, LIBRARY],
                             input=json.dumps(calls), capture_output=True, text=True, timeout=300)
        assert res.returncode == 0, res.stderr[-3000:]
        return json.loads(res.stdout)
    return run


# layers, blocks, block_size, heads, head_dim: tiles of 8 and 64 KiB
SMALL, LARGE = (4, 2000, 16, 2, 128), (11, 64, 32, 8, 128)


@pytest.mark.parametrize("call", ["pack", "unpack"])
@pytest.mark.parametrize("pool", [SMALL, LARGE], ids=["8KiB", "64KiB"])
def test_host_staging_copies_move_one_row_a_wavefront(record, call, pool):
    """Few rows or many, a copy to or from host memory takes one 1 KiB row per
    wavefront: two rows slow small transfers over the link."""
    tile = pool[2] * pool[3] * pool[4] * 2
    for n in (1, 5, 60):
        got = record([dict(call=call, pool_args=pool, blocks=list(range(n)), staging="host")])[0]
        assert got["rc"] == 0
        (one,) = got["launches"]
        assert one["kernel"] == "copy_rows" and one["template"][3] == 1 and one["block"] == 64
        assert one["grid"] == one["items"] == n * 2 * pool[0] * tile // 1024


@pytest.mark.parametrize("call", ["stage", "pack", "unpack"])
def test_small_copies_move_two_rows_a_wavefront(record, call):
    """On the GPU, up to one round of resident wavefronts (8192 rows), and in
    workgroups of two wavefronts, which every item fills."""
    where = [dict(src=list(range(n)), dst=list(range(n))) if call == "stage" else
             dict(blocks=list(range(n)), staging="device") for n in (32, 33)]
    one, two = record([dict(call=call, pool_args=(1, 64, 16, 32, 128), **w) for w in where])
    assert one["launches"][0]["template"][3] == 2 and two["launches"][0]["template"][3] == 1
    assert one["launches"][0]["items"] == 32 * 2 * 64 and two["launches"][0]["items"] == 33 * 2 * 128
    assert (one["launches"][0]["grid"], one["launches"][0]["block"]) == (32 * 64, 128)
    assert (two["launches"][0]["grid"], two["launches"][0]["block"]) == (33 * 2 * 128, 64)
    # tiles of an odd number of KiB and less than one: still whole workgroups
    for pool in ((1, 64, 8, 1, 64), (3, 64, 8, 3, 64), (1, 64, 16, 3, 128)):
        for w in where:
            for x in record([dict(call=call, pool_args=pool, **w)])[0]["launches"]:
                assert x["block"] == 128 and x["grid"] * 2 == x["items"]


def pairs_of(launches):
    """The (source, destination) pairs of a call in launch order, and the place
    of a staging source where pairs carry one."""
    out, seen = [], set()
    for x in launches:
        if x.get("lin_first") in seen:          # a later slice of the same pairs
            continue
        seen.add(x["lin_first"])
        for k in range(x["pairs"]):
            out.append((x["ids"][k] & 0xffff, x["ids"][k] >> 16) if x["template"][2 if x["kernel"] == "copy_rows" else 0] == 2
                       else (x["ids"][k], x["ids"][256 + k]))
    return out


def in_order(dst, top):
    """Ascending in the leading 11 bits of the largest id's bits."""
    shift = max(0, int(top).bit_length() - 11)
    d = np.asarray(dst) >> shift
    return bool((np.diff(d) >= 0).all())


# pool, pairs, whether ordering them by destination pays: under 32 pairs; 48 MiB
# one way or less, of any tile; pairs of less than 64 KiB; thousands of pairs
ORDER = [((32, 6000, 16, 32, 128), 31, False), ((32, 6000, 16, 32, 128), 32, True),
         ((1, 6000, 16, 32, 128), 191, False), ((1, 6000, 16, 32, 128), 192, True),
         ((1, 6000, 16, 1, 128), 5000, False), ((8, 6000, 16, 1, 128), 767, False),
         ((8, 6000, 16, 1, 128), 768, True), ((7, 70000, 16, 1, 128), 5000, False),
         ((8, 70000, 16, 1, 128), 5000, True)]


@pytest.mark.parametrize("call", ["stage", "convert", "unpack", "unpack_layout"])
def test_pairs_are_ordered_only_where_it_pays(record, call):
    g = np.random.default_rng(5)
    calls, want = [], []
    for pool, n, _ in ORDER:
        src, dst = (g.permutation(pool[1])[:n].tolist() for _ in range(2))
        if call in ("stage", "convert"):
            calls.append(dict(call="stage", pool_args=pool, src=src, dst=dst,
                              layouts=((0, 0), (0, 0) if call == "stage" else (1, 1))))
        else:
            src = list(range(n))                # places in the staging buffer
            calls.append(dict(call=call, pool_args=pool, blocks=dst, staging="device"))
            if call == "unpack_layout":
                calls[-1]["staging_layouts"] = (1, 1)
        want.append((src, dst))
    for (pool, n, ordered), got, (src, dst) in zip(ORDER, record(calls), want):
        assert got["rc"] == 0
        pairs = pairs_of(got["launches"])
        assert sorted(pairs) == sorted(zip(src, dst)), (pool, n)
        if ordered:
            assert in_order([d for _, d in pairs], max(dst)), (pool, n)
        else:
            assert pairs == list(zip(src, dst)), (pool, n)


# pool, layouts, first token, tokens, the kernel that writes them
WRITES = [((80, 300, 16, 32, 128), (0, 0), 3, 64, "write_token_slots"),     # appends, whatever their bytes
          ((1, 300, 16, 8, 128), (0, 0), 3, 65, "write_rows"),
          ((80, 300, 16, 8, 128), (0, 0), 0, 4800, "write_rows"),
          ((2, 300, 16, 7, 128), (0, 0), 0, 1, "write_rows"),               # slots under 2 KiB
          ((2, 300, 16, 8, 128), (2, 3), 0, 1, "write_token_slots"),
          ((2, 300, 16, 8, 128), (2, 3), 15, 2, "write_slabs"),
          ((2, 300, 16, 8, 128), (0, 1), 0, 4700, "write_slabs"),
          ((2, 300, 12, 8, 128), (2, 3), 0, 100, "write_token_slots"),      # HDN, 8 does not divide the block
          ((2, 300, 256, 8, 128), (1, 1), 0, 100, "write_token_slots")]     # slabs over 16 KiB


def test_token_writes(record):
    """The kernel of a write, and that its launches cover every token once."""
    for (pool, layouts, first, n, kernel), got in zip(WRITES, record([
            dict(call="write", pool_args=p, table=list(range(300)), first=f, tokens=n, layouts=l) for p, l, f, n, _ in WRITES])):
        assert got["rc"] == 0 and {x["kernel"] for x in got["launches"]} == {kernel}, (pool, layouts, n)
        at = 0
        for x in got["launches"]:
            assert x["lin_first" if kernel == "write_slabs" else "first_token"] == at
            assert x["first_slot"] == (first + at) % pool[2]
            blocks = x["pairs" if kernel == "write_slabs" else "blocks"]
            assert blocks == (first + at + x["tokens"] - 1) // pool[2] - (first + at) // pool[2] + 1 <= 256
            assert x["ids"][:blocks] == list(range((first + at) // pool[2], (first + at) // pool[2] + blocks))
            if kernel == "write_rows":
                run = min(pool[2], x["tokens"]) * x["slot_bytes"]
                assert x["rows_per_run"] == -(-run // 1024) and x["grid"] == blocks * 2 * pool[0] * x["rows_per_run"]
            elif kernel == "write_slabs":
                assert x["grid"] == blocks * 2 * pool[0] * pool[3]
            at += x["tokens"]
        assert at == n


# ---- decode attention ---------------------------------------------------------

def partitions(launches):
    """{sequence: [(first token, end)]} of a call as its kernels will number
    them, and its workgroups, checked: sequences of several partitions come
    first, longest partition first (after a sequence that carries a stage and is
    launched apart), launches cover every item once, and the merge reads the
    records the partial kernel leaves."""
    partial = [x for x in launches if x["kernel"] == "attn_partial_mfma"]
    a = partial[0]
    per_item = a["kv_heads"] * a["num_layers"]
    out, first, lengths = {}, 0, []
    for s in range(a["batch"]):
        end, n = a["item_end"][s], a["ctx"][s]
        word = a["seq"][s // 2] >> (16 * (s % 2))
        b, plen = word & 0xff, (word >> 8 & 0xff) * 64
        parts = end - first
        assert b not in out and parts >= 1
        if parts == 1:
            out[b] = [(0, n)]
        else:
            out[b] = [(i * plen, min(n, (i + 1) * plen)) for i in range(parts)]
            assert out[b][-1][0] < n <= parts * plen
        lengths.append((parts == 1, -(plen if parts > 1 else n)))
        assert max(e - t for t, e in out[b]) <= a["part_tokens"] <= 2048
        first = end
    apart = len({x["template"][2] for x in partial}) == 2
    assert lengths[apart:] == sorted(lengths[apart:]) and lengths[0][0] <= lengths[-1][0]
    assert a["n_records"] == sum(len(p) for p in out.values() if len(p) > 1)
    items, at = first, 0
    for x in partial:
        assert x["item_base"] == at and x["grid"] % per_item == 0 and x["grid"] // per_item >= 1
        assert x["grid"] <= 1 << 22 or x["grid"] == per_item
        at += x["grid"] // per_item
    assert at == items
    merge = [x for x in launches if x["kernel"] == "attn_reduce"]
    several = [b for b in out if len(out[b]) > 1]
    assert bool(merge) == bool(several)
    if merge:
        m = merge[0]
        assert m["seqs"] == len(several) and m["seq"][:len(several)] == several
        assert np.diff([0] + m["seq_end"][:len(several)]).tolist() == [len(out[b]) for b in several]
        rows, per_wg = m["num_layers"] * m["seqs"] * m["q_heads"], 256 // (m["head_dim"] // 4) if m["template"][1] == 1 else 1
        assert m["template"][1] > 1 or max(len(p) for p in out.values()) <= 8
        at = 0
        for x in merge:
            assert x["row_base"] == at and x["grid"] <= 1 << 22
            at += x["grid"] * per_wg
        assert rows <= at < rows + per_wg
    return out, items * per_item


def decode(pool, ctx, group=1, workspace="full", carry=None, seq=0):
    return dict(call="decode", pool_args=pool, ctx=ctx, group=group, workspace=workspace, carry=carry, seq=seq)


def test_attention_partitions_cover_every_token(record):
    """Random calls, batches up to 256, empty sequences among them."""
    g = np.random.default_rng(7)
    calls = []
    for k in range(60):
        batch = int(g.choice([1, 3, 17, 64, 255, 256]))
        pool = (int(g.integers(1, 5)), 8, int(g.choice([1, 12, 16, 32])), int(g.choice([1, 4, 8])), int(g.choice([64, 128])))
        ctx = np.exp(g.uniform(0, np.log(int(g.choice([500, 3000, 40000]))), batch)).astype(int)
        ctx[g.random(batch) < 0.1] = 0
        calls.append(decode(pool, ctx.tolist(), int(g.choice([1, 4, 16])), ["full", "least"][k % 2]))
    for c, got in zip(calls, record(calls)):
        assert got["rc"] == 0, c
        parts, _ = partitions(got["launches"])
        for b, n in enumerate(c["ctx"]):
            assert parts[b][0][0] == 0 and parts[b][-1][1] == n
            assert all(x[1] == y[0] and y[0] % 64 == 0 for x, y in zip(parts[b], parts[b][1:]))
        layers, _, _, heads, dim = c["pool_args"]
        assert [parts[b] for b in range(len(c["ctx"]))] == attn_cases.partitions(c["ctx"], layers, heads, dim,
                                                                                 c["workspace"])


def test_attention_runs_as_several_launches(record):
    """A launch holds 2^22 workgroups: 256 items of 128 layers of 128 heads, and
    as many rows of the merge (16 a workgroup for head_dim 64)."""
    got, wide = record([decode((128, 8, 16, 128, 64), [5000] * 256), decode((160, 8, 16, 128, 64), [5000] * 256, 16)])
    _, workgroups = partitions(got["launches"])
    assert workgroups == 256 * 3 * 128 * 128 and [x["kernel"] for x in got["launches"]] == ["attn_partial_mfma"] * 3 + ["attn_reduce"]
    partitions(wide["launches"])
    assert sum(x["kernel"] == "attn_reduce" for x in wide["launches"]) == 2


# one layer of 8 heads unless said: calls that fill the chip in whole partitions
# of 2048, or whose sequences are short, are cut no further
UNCUT = [((1, 8, 16, 8, 128), [1000, 200] * 32), ((1, 8, 16, 8, 64), [1000, 200] * 32),
         ((1, 8, 16, 8, 128), [768]), ((8, 8, 16, 8, 128), [1364] * 9), ((4, 8, 16, 8, 64), [1439] * 17),
         ((1, 8, 16, 32, 64), [13646] * 4), ((1, 8, 16, 32, 128), [22639] * 3),
         ((32, 8, 16, 8, 128), [962, 500, 400])]


@pytest.mark.parametrize("workspace", ["full", "none"])
def test_attention_is_not_cut_past_a_full_chip(record, workspace):
    for (pool, ctx), got in zip(UNCUT, record([decode(p, c, 1, workspace) for p, c in UNCUT])):
        parts, _ = partitions(got["launches"])
        assert all(len(parts[b]) == max(1, -(-n // 2048)) for b, n in enumerate(ctx)), (pool, ctx)


def test_attention_cuts_fill_the_chip_and_no_more(record):
    """Short of workgroups, a call is cut to at most two a CU (one for sequences
    over 2048 tokens of head_dim 128), where the merge is needed anyway to the
    next whole number up to three, and to no fewer than half of that unless
    partitions reach 256 tokens."""
    g = np.random.default_rng(11)
    calls = []
    for _ in range(80):
        pool = (int(g.choice([1, 1, 2, 4])), 8, 16, int(g.choice([1, 2, 4, 8])), int(g.choice([64, 128])))
        calls.append(decode(pool, np.exp(g.uniform(np.log(769), np.log(30000), int(g.integers(1, 9)))).astype(int).tolist(), 4))
    cut = 0
    for c, got in zip(calls, record(calls)):
        (layers, _, _, heads, dim), ctx = c["pool_args"], c["ctx"]
        parts, workgroups = partitions(got["launches"])
        whole = layers * heads * sum(-(-n // 2048) for n in ctx)
        if all(len(parts[b]) <= -(-n // 2048) for b, n in enumerate(ctx)):
            continue
        cut += 1
        most = 512 if dim == 64 or max(ctx) <= 2048 else 256
        if max(ctx) > 2048:
            most = max(most, min(768, -(-whole // 256) * 256))
        assert whole <= most and workgroups <= most, c
        longest = max(e - t for p in parts.values() for t, e in p)
        assert longest == 256 or workgroups >= most // 2, (c, workgroups, longest)
        assert longest <= (0.9 if max(ctx) > 2048 else 0.75) * min(2048, max(ctx)) + 63
    assert cut > 30


def test_attention_of_the_smaller_workspace_has_partitions_of_2048(record):
    pool, ctx = (1, 8, 16, 8, 128), [3000, 900, 700, 0]
    full, least = record([decode(pool, ctx, 4, w) for w in ("full", "least")])
    assert len(partitions(full["launches"])[0][0]) > 2
    assert [len(partitions(least["launches"])[0][b]) for b in range(4)] == [2, 1, 1, 1]


# pool, lengths, workgroups a CU that the launch leaves room for (0: no limit)
ROOM = [((8, 8, 16, 13, 64), [17400] * 1 + [4000], 0),          # 1144: a second round of a few would lose
        ((32, 8, 16, 13, 64), [8000], 4), ((32, 8, 16, 13, 128), [8000], 3),
        ((1, 8, 16, 13, 128), [16000] * 10, 0), ((4, 8, 16, 8, 128), [16000] * 5, 3),
        ((1, 8, 16, 8, 64), [14000] * 16, 2), ((1, 8, 16, 8, 128), [14000] * 16, 2),
        ((1, 8, 16, 8, 64), [12000] * 16, 0),                   # 768
        ((1, 8, 12, 8, 64), [14000] * 16, 2),                   # block ids in LDS beside it
        ((32, 8, 16, 32, 64), [700] * 8, 0), ((32, 8, 16, 32, 128), [1400] * 8, 0)]


def test_attention_of_long_partitions_leaves_room(record):
    static = {64: 17920, 128: 34304}
    for (pool, ctx, want), got in zip(ROOM, record([decode(p, c) for p, c, _ in ROOM])):
        parts, workgroups = partitions(got["launches"])
        lds = got["launches"][0]["lds"]
        if want == 0:
            assert lds == 0, (pool, ctx, workgroups)
        else:
            assert 163840 // (static[pool[4]] + lds) == want, (pool, ctx, workgroups, lds)
    # carrying a stage: by the length of the partitions alone, and cut as the plain call
    calls = [((4, 2000, 16, 32, 64), [16528], 4), ((4, 2000, 16, 8, 128), [16000] * 4, 3), ((1, 2000, 16, 8, 64), [700], 0)]
    for (pool, ctx, want), got, plain in zip(calls, record([decode(p, c, carry=9) for p, c, _ in calls]),
                                             record([decode(p, c) for p, c, _ in calls])):
        lds = got["launches"][0]["lds"]
        assert got["rc"] == 0 and (163840 // (static[pool[4]] + lds) if lds else 0) == want
        assert partitions(got["launches"]) == partitions(plain["launches"])


def test_many_short_sequences_of_head_dim_64_run_layer_by_layer(record):
    calls = [((128, 8, 16, 32, 64), [20] * 2, True), ((127, 8, 16, 32, 64), [20] * 2, False),
             ((128, 8, 16, 32, 64), [199] * 2, True), ((128, 8, 16, 32, 64), [200] * 2, False),
             ((128, 8, 16, 32, 128), [20] * 2, False), ((256, 8, 16, 256, 64), [20] * 200, True)]
    for (pool, ctx, want), got in zip(calls, record([decode(p, c) for p, c, _ in calls])):
        partitions(got["launches"])
        for x in got["launches"]:
            assert x["layer_items"] == (x["grid"] // (pool[0] * pool[3]) if want else 0)
    # not a launch that carries a stage
    (got,) = record([decode((128, 8, 16, 32, 64), [20] * 2, carry=1)])
    assert got["rc"] == 0 and [x["layer_items"] for x in got["launches"]] == [0]


# pool, lengths, the sequence whose blocks are carried, whether it is launched apart
APART = [((40, 300, 16, 20, 128), [30] * 19 + [41], 7, True), ((40, 300, 16, 20, 128), [30] * 18 + [41], 7, False),
         ((40, 300, 16, 20, 64), [30] * 19 + [41], 19, True), ((40, 300, 16, 20, 64), [30] * 18 + [41], 0, False),
         ((40, 300, 16, 20, 128), [159] * 20, 0, True), ((40, 300, 16, 20, 128), [160] * 20, 0, False),
         ((200, 300, 12, 100, 128), [30], 0, False),                    # alone
         ((80, 300, 16, 4, 128), [5, 0, 17] * 30 + [4097, 2100], 91, True),     # cut, after a longer one
         ((80, 300, 16, 4, 128), [5, 0, 17] * 30 + [4097, 2100], 90, True),
         ((80, 300, 16, 4, 128), [5, 0, 17] * 30 + [4097, 2100], 0, False),     # whole, beside cut ones
         ((256, 300, 16, 256, 64), [20] * 200, 199, True)]              # several launches of the others


def test_the_sequence_a_call_of_many_short_ones_carries_is_launched_apart(record):
    for (pool, ctx, seq, apart), got, plain in zip(APART, record([decode(p, c, carry=1, seq=s) for p, c, s, _ in APART]),
                                                   record([decode(p, c) for p, c, _, _ in APART])):
        what = (pool, ctx[:3], seq)
        assert got["rc"] == 0, what
        parts, workgroups = partitions(got["launches"])
        assert (parts, workgroups) == partitions(plain["launches"]), what
        per_item = pool[0] * pool[3]
        partial = [x for x in got["launches"] if x["kernel"] == "attn_partial_mfma"]
        carrying = [x for x in partial if x["template"][2] == 1]
        assert all(x["mig_seq"] == seq and x["template"][3] == (pool[2] % 8 == 0) for x in partial), what
        if apart:
            assert partial[0] is carrying[0] and len(carrying) == 1 and len(partial) >= 2, what
            assert carrying[0]["grid"] == len(parts[seq]) * per_item and list(parts)[0] == seq, what
            assert carrying[0]["layer_items"] == 0, what
            assert all(x["layer_items"] == (x["grid"] // per_item if pool[4] == 64 else 0) for x in partial[1:]), what
        else:
            assert len(carrying) == len(partial), what

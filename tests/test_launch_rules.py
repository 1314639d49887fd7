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
    """On the GPU, up to one round of resident wavefronts (8192 rows)."""
    where = [dict(src=list(range(n)), dst=list(range(n))) if call == "stage" else
             dict(blocks=list(range(n)), staging="device") for n in (32, 33)]
    one, two = record([dict(call=call, pool_args=(1, 64, 16, 32, 128), **w) for w in where])
    assert one["launches"][0]["template"][3] == 2 and one["launches"][0]["grid"] == 32 * 2 * 64
    assert two["launches"][0]["template"][3] == 1 and two["launches"][0]["grid"] == 33 * 2 * 128


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

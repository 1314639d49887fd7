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
def test_staging_copies_move_one_row_a_wavefront(record, call, pool):
    """Few rows or many, a copy to or from a staging buffer takes one 1 KiB row
    per wavefront: two rows would slow small transfers over the host link."""
    tile = pool[2] * pool[3] * pool[4] * 2
    for n in (1, 5, 60):
        got = record([dict(call=call, pool_args=pool, blocks=list(range(n)), staging="host")])[0]
        assert got["rc"] == 0
        (one,) = got["launches"]
        assert one["kernel"] == "copy_rows" and one["template"][3] == 1 and one["block"] == 64
        assert one["grid"] == one["items"] == n * 2 * pool[0] * tile // 1024


def test_small_stages_move_two_rows_a_wavefront(record):
    """Pool to pool, up to one round of resident wavefronts (8192 rows)."""
    one, two = record([dict(call="stage", pool_args=(1, 64, 16, 32, 128), src=list(range(n)), dst=list(range(n)))
                       for n in (32, 33)])
    assert one["launches"][0]["template"][3] == 2 and one["launches"][0]["grid"] == 32 * 2 * 64
    assert two["launches"][0]["template"][3] == 1 and two["launches"][0]["grid"] == 33 * 2 * 128

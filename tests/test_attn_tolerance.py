"""The decode-attention error bound can fail (CPU only).

The GPU parity test accepts the kernel's output when it lies within the
bound of tests/attn_cases.py of the fp64 oracle.  A bound that grows with
the sequence length alone would also accept an output that lost a whole
partition of a long sequence, or the later half of a call's partitions,
which is exactly the kind of mistake a flash-decoding merge can make.  Here,
for every fixed case cut as the library cuts it, the oracle's own result
with such a piece dropped must violate the bound, while the exact result
passes it with room to spare."""
import numpy as np
import pytest

import attn_cases as ac


def _oracle_and_bound(case, workspace="full"):
    host, q, tables, ctx, scale = ac.case_inputs(case, ac.case_seed(case))
    _, _, bs, kv_heads, head_dim, _, _, dtype, _ = case
    orc = ac.default_oracle()
    want = orc.decode_attention(host, kv_heads, head_dim, dtype, q, tables, ctx, scale)
    tol = ac.tolerance(orc, host, kv_heads, head_dim, dtype, q, tables, ctx, scale, workspace)
    return orc, host, q, tables, ctx, scale, want, tol


def _dropped(orc, case, host, q, tables, ctx, scale, pieces):
    """Oracle output with the token ranges pieces[b] = [(lo, hi), ...] removed."""
    _, _, bs, kv_heads, head_dim, _, _, dtype, _ = case
    t, n = tables, list(ctx)
    for b, ranges in pieces.items():
        for lo, hi in sorted(ranges, reverse=True):        # later ranges first: earlier offsets stay valid
            t, n = ac.drop_tokens(t, n, bs, b, lo, hi)
    return orc.decode_attention(host, kv_heads, head_dim, dtype, q, t, n, scale)


def _partitions(case, workspace="full"):
    return ac.partitions(case[6], case[0], case[3], case[4], workspace)


# cases with a sequence of several partitions whose edges are block edges; the
# largest, whose oracle calls take seconds each, is the second test's
MULTI = [c for c in ac.CASES if 64 % c[2] == 0 and max(len(p) for p in _partitions(c)) > 1]


@pytest.mark.parametrize("workspace", ["full", "least"])
@pytest.mark.parametrize("case", [c for c in MULTI if max(c[6]) <= 50000], ids=ac.case_id)
def test_dropping_one_partition_violates_the_bound(case, workspace):
    orc, host, q, tables, ctx, scale, want, tol = _oracle_and_bound(case, workspace)
    assert ac.excess(want, want, tol).max() == 0.0
    for b, parts in enumerate(_partitions(case, workspace)):
        if len(parts) < 2:
            continue
        for j in sorted({0, len(parts) // 2, len(parts) - 1}):
            got = _dropped(orc, case, host, q, tables, ctx, scale, {b: [parts[j]]})
            ratio = ac.excess(got[:, b], want[:, b], tol[:, b]).max()
            print(f"sequence {b} ({ctx[b]} tokens), partition {j} of {len(parts)} {parts[j]} dropped: "
                  f"max error / bound {ratio:.3g}")
            assert ratio > 1.0, f"sequence {b}: dropping partition {j} stays within the bound"


@pytest.mark.parametrize("case", [c for c in MULTI if max(c[6]) > 50000], ids=ac.case_id)
def test_dropping_the_later_partitions_violates_the_bound(case):
    """What a launch lost from the middle of a call on would cost."""
    orc, host, q, tables, ctx, scale, want, tol = _oracle_and_bound(case)
    pieces = {b: [(parts[len(parts) // 2][0], ctx[b])] for b, parts in enumerate(_partitions(case)) if len(parts) > 1}
    got = _dropped(orc, case, host, q, tables, ctx, scale, pieces)
    for b in pieces:
        ratio = ac.excess(got[:, b], want[:, b], tol[:, b]).max()
        print(f"later half dropped: sequence {b}, max error / bound {ratio:.3g}")
        assert ratio > 1.0


def test_bound_is_small_against_the_output():
    """Where the weighted mean of |V| is not tiny (a one-token row can make
    it so, and then the absolute terms dominate), the bound is a small
    fraction of it: under 5e-4, about 1.5e-4 at 50,000 tokens."""
    for case in ac.CASES:
        orc, host, q, tables, ctx, scale, want, tol = _oracle_and_bound(case)
        A = orc.decode_attention(ac.abs_v_pool(host), case[3], case[4], case[7], q, tables, ctx, scale)
        live = A > 0.05
        rel = (tol[live] / A[live]).max()
        print(f"{ac.case_id(case)}: largest bound / weighted |V| = {rel:.3g}")
        assert rel < 5e-4


def test_drop_tokens_is_attention_over_the_rest():
    """drop_tokens keeps every other token: on a small case, dropping a
    range equals attention over a table and length built by hand."""
    case = (1, 64, 4, 1, 64, 2, [40], "fp16", False)
    host, q, tables, ctx, scale = ac.case_inputs(case, 7)
    orc = ac.default_oracle()
    t, n = ac.drop_tokens(tables, ctx, 4, 0, 8, 20)
    assert n == [28]
    by_hand = np.zeros_like(tables)
    row = list(tables[0, :2]) + list(tables[0, 5:10])
    by_hand[0, :len(row)] = row
    a = orc.decode_attention(host, 1, 64, "fp16", q, t, n, scale)
    b = orc.decode_attention(host, 1, 64, "fp16", q, by_hand, [28], scale)
    assert np.array_equal(a, b)
    full = orc.decode_attention(host, 1, 64, "fp16", q, tables, ctx, scale)
    assert not np.array_equal(a, full)

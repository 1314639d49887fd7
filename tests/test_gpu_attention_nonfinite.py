"""Decode attention on scores that are not finite.

A row (layer, sequence, query head) with a NaN score gives zeros, however the
call is cut: whole sequences, partitions of 2048 tokens and of 256, partitions
that hold nothing but NaN scores.  Scores of -inf (keys near the lowest bf16
value, whose products with the query overflow) are weights of 0, also where a
partition or a wavefront's share of it starts with them; a row of nothing else
gives zeros.  Reference: torch's softmax in float64, rows with NaN scores and
rows of -inf set to 0."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2406_03243_amd.llmig import (Pool, decode_workspace_bytes, llmig_decode_attention,
                                            llmig_decode_attention_noalloc)

LOWEST = -3.38e38           # a bf16 key whose product with a query element of 4 is -inf in fp32

# block_size, head_dim, layers, kv_heads, length; the first two call shapes are
# whole, the third is cut finely, the fourth (and any with the smaller
# workspace) into partitions of 2048
SHAPES = [(16, 128, 1, 2, 300), (12, 64, 2, 1, 500), (16, 64, 1, 2, 2500), (16, 128, 8, 16, 4500)]


def spans(n):
    """(name, first token, last token + 1) of the tokens whose score is set."""
    return [("first", 0, 1), ("first_group", 0, 64), ("first_part", 0, min(n, 256)), ("middle", n // 2, n // 2 + 1),
            ("second_wave", 16, 32), ("tail", n - 70, n), ("late_part", min(n - 1, 2048), min(n, 2304)), ("all", 0, n)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"bs{s[0]}_D{s[1]}_L{s[2]}_n{s[4]}")
@pytest.mark.parametrize("bad", ["nan", "-inf"])
def test_nonfinite_scores(shape, bad):
    bs, dim, layers, heads, n = shape
    group = 2
    names = spans(n)
    batch, blocks = len(names), -(-n // bs)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    kv = torch.empty((2, layers, batch * blocks, bs, heads, dim), dtype=torch.bfloat16, device="cuda")
    kv.normal_(generator=gen)
    q = torch.empty((layers, batch, heads * group, dim), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q[..., 0] = 4.0
    kv[0, ..., 0] = 0.0
    tables = torch.randperm(batch * blocks, generator=gen, device="cuda").to(torch.int32).view(batch, blocks)
    for b, (_, lo, hi) in enumerate(names):     # of KV head 0 only
        t = torch.arange(lo, hi, device="cuda")
        kv[0, :, tables[b].long()[t // bs], t % bs, 0, 0] = float("nan") if bad == "nan" else LOWEST
    pool = Pool(list(kv[0].unbind(0)), list(kv[1].unbind(0)))
    scale, lens = 1.0 / math.sqrt(dim), [n] * batch
    want = torch.zeros(q.shape, dtype=torch.float64)
    for layer in range(layers):
        for b in range(batch):
            k, v = (kv[j, layer, tables[b].long()].reshape(-1, heads, dim)[:n].double().cpu() for j in (0, 1))
            for h in range(heads * group):
                s = (k[:, h // group] @ q[layer, b, h].double().cpu()) * scale
                if bad == "-inf":
                    s[s < -1e30] = -math.inf
                if not bool(torch.isnan(s).any()) and bool(torch.isfinite(s).any()):
                    want[layer, b, h] = torch.softmax(s, 0) @ v[:, h // group]
    full = decode_workspace_bytes(lens, layers, heads * group, dim)
    least = layers * heads * group * batch * -(-n // 2048) * (dim + 4) * 4
    for name, nbytes in (("returned size", full), ("smallest size", least), ("no workspace", 0)):
        print("[case]", shape, bad, name, flush=True)
        out = torch.full(q.shape, 7.0, dtype=torch.float32, device="cuda")
        if nbytes:
            ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
            llmig_decode_attention(pool, q, tables, lens, scale, ws, out)
        else:
            llmig_decode_attention_noalloc(pool, q, tables, lens, scale, out)
        torch.cuda.synchronize()
        got = out.double().cpu()
        assert bool(torch.isfinite(got).all()), [names[i][0] for i in np.unique(np.argwhere(~np.isfinite(got.numpy()))[:, 1])]
        # unit normal values: fp32 sums of weights that carry 2^-16
        assert float((got - want).abs().max()) < 1e-3
        assert bool((got[want.abs().sum(-1) == 0] == 0).all())

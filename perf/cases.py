"""The work a serving system has this framework do, as cases that can be timed
and compared: whole migrations, single stages, block fusion, decode attention
and the KV writes beside it, each through the public entry points.

A case is a dict of plain values.  ``kind`` names the call; ``layers``,
``heads`` (KV heads of this GPU's shard), ``dim``, ``block`` (tokens per
block) and ``dtype`` give the pool.  ``listed()`` holds the fixed cases,
``draw(rng)`` one more of the same ranges, ``prepare`` what a program has in
hand before the call, ``run`` one pass through it, ``work`` the bytes and
operations a pass cannot do without, ``tolerance`` and ``exact`` what its
result is held to.

Copies and writes move bytes, so their outputs are compared as raw 16-bit
words; decode attention computes, in fp32 from 16-bit inputs, and is compared
with a float64 evaluation.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2406_03243_amd import harness, migrate
from paper_2406_03243_amd import llmig

DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16}
LAYOUTS = {"NHD": llmig.LAYOUT_NHD, "HND": llmig.LAYOUT_HND, "HCNX": llmig.LAYOUT_HCNX, "HDN": llmig.LAYOUT_HDN}


def listed():
    return [
        # A 7B-shaped request of 8k tokens leaves its instance while decoding
        # goes on: one long stage, three short ones, the final stage.
        dict(name="migrate_multistage", kind="migrate", layers=32, heads=32, dim=128, block=16, dtype="fp16",
             tokens=8192, batches=4, append=37),
        # A request that has only just started is moved at once: one block,
        # all of it downtime (one tensor-parallel rank of a 30B shape).
        dict(name="migrate_short", kind="finish", layers=60, heads=13, dim=128, block=16, dtype="fp16", tokens=11),
        # Several requests of a drained instance in one call.
        dict(name="stage_batched", kind="stage", layers=32, heads=32, dim=128, block=16, dtype="bf16", pairs=487,
             ids="host", layouts="NHD/NHD>NHD/NHD"),
        # A long request of a grouped-query model on one rank of eight: a
        # single KV head, so tiles of 4 KiB.
        dict(name="stage_one_head", kind="stage", layers=80, heads=1, dim=128, block=16, dtype="bf16", pairs=2048,
             ids="host", layouts="NHD/NHD>NHD/NHD"),
        # Between two engines that keep their tiles in different orders.
        dict(name="stage_cross_layout", kind="stage", layers=32, heads=32, dim=128, block=16, dtype="fp16", pairs=256,
             ids="host", layouts="NHD/NHD>HCNX/HDN"),
        # Block fusion on one GPU: gather into a staging buffer, scatter from it.
        dict(name="pack_unpack", kind="fuse", layers=60, heads=13, dim=128, block=16, dtype="fp16", pairs=253,
             ids="host", layouts="NHD/NHD>NHD/NHD"),
        # Block fusion through pinned host memory, both directions at once.
        dict(name="host_staged", kind="host", layers=80, heads=8, dim=128, block=16, dtype="bf16", pairs=64, chunk=16),
        # One decode step of a grouped-query batch, all layers in one call.
        dict(name="decode_gqa", kind="decode", layers=80, heads=8, dim=128, block=16, dtype="bf16", group=8, batch=16,
             ctx=4096, call="workspace"),
        # One layer of a small batch, as a model calls it layer by layer
        # from code that cannot allocate.
        dict(name="decode_one_layer", kind="decode", layers=1, heads=8, dim=128, block=16, dtype="bf16", group=4,
             batch=3, ctx=3000, call="noalloc"),
        # One decode step of a 7B-shaped batch: a query head per KV head.
        dict(name="decode_mha", kind="decode", layers=32, heads=32, dim=128, block=16, dtype="fp16", group=1, batch=8,
             ctx=1500, call="workspace"),
        # A decode step that carries the first stage of one of its requests.
        dict(name="decode_carrying", kind="decode", layers=80, heads=8, dim=128, block=16, dtype="bf16", group=8,
             batch=6, ctx=8000, call="carry"),
        # A prompt's keys and values are written in the paged layouts.
        dict(name="write_prompt", kind="write", layers=32, heads=32, dim=128, block=16, dtype="fp16", requests=1,
             tokens=2000, first=0, layouts="HCNX/HDN"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random) -> dict:
    """One more case: any kind, with a pool of a shape that models and their
    tensor-parallel shards have, and sizes spread over the logarithm of the
    range; none is costlier than the largest listed case."""
    kind = rng.choice(["migrate", "finish", "stage", "stage", "stage", "fuse", "host", "decode", "decode", "decode",
                       "decode", "write", "write"])
    heads = rng.choice([1, 2, 4, 8, 8, 13, 32, 32, rng.randint(1, 40)])
    c = dict(kind=kind, layers=_log_int(rng, 1, 80), heads=heads, dim=rng.choice([64, 128, 128]),
             block=rng.choice([8, 16, 16, 16, 32]), dtype=rng.choice(["fp16", "bf16"]))
    per_block = c["layers"] * 2 * c["block"] * heads * c["dim"] * 2
    per_token = per_block // c["block"]
    converts = ["NHD/NHD>HND/HND", "NHD/NHD>HCNX/HDN", "HCNX/HDN>NHD/NHD", "HND/HND>NHD/NHD", "HND/HND>HCNX/HDN",
                "NHD/HND>NHD/NHD"]
    if kind == "migrate":
        c.update(batches=rng.randint(1, 5), append=rng.randint(1, 64))
        most = max(2, min(16384, 3_600_000_000 // per_token))
        c["tokens"] = _log_int(rng, min(64, most // 2), most)
    elif kind == "finish":
        c["tokens"] = _log_int(rng, 1, max(2, min(600, 300_000_000 // per_token)))
    elif kind in ("stage", "fuse"):
        most = max(2, min(4096, (3_600_000_000 if kind == "stage" else 1_800_000_000) // per_block))
        c.update(pairs=_log_int(rng, 1, most), ids=rng.choice(["host", "host", "device"]),
                 layouts=rng.choice(["NHD/NHD>NHD/NHD", "HND/HND>HND/HND", rng.choice(converts)]))
    elif kind == "host":
        c["pairs"] = _log_int(rng, 1, max(2, min(512, 300_000_000 // per_block)))
        c["chunk"] = max(1, c["pairs"] // rng.randint(1, 6))
    elif kind == "decode":
        c.update(group=rng.choice([1, 2, 4, 8, 8, 16]), batch=_log_int(rng, 1, 64),
                 call=rng.choice(["workspace", "workspace", "noalloc", "carry"]))
        if c["heads"] * c["group"] > 128:
            c["group"] = 1
        if c["call"] == "noalloc":
            c["layers"], per_token = 1, per_token // c["layers"]
        most = max(64, min(32768, 6_000_000_000 // per_token // c["batch"]))
        if c["call"] == "noalloc":        # what its static scratch holds
            most = min(most, 400_000 // c["batch"])
        c["ctx"] = _log_int(rng, 32, most)
    else:
        c.update(layouts=rng.choice(["NHD/NHD", "HND/HND", "HCNX/HDN", "HCNX/HDN"]), requests=rng.choice([1, 1, 4, 16]))
        most = max(2, min(4096, 1_000_000_000 // per_token // c["requests"]))
        c["tokens"] = rng.choice([1, rng.randint(1, 8), _log_int(rng, 1, most)])
        c["tokens"] = min(c["tokens"], most)
        c["first"] = rng.choice([0, rng.randint(0, 200)])
    return c


# ---- what a case comes to ---------------------------------------------------

def _tile(c):
    return c["block"] * c["heads"] * c["dim"] * 2


def _blocks(c, tokens):
    return -(-tokens // c["block"])


def _context_lengths(c):
    """Lengths of a decode batch: the longest is ``ctx``, the others spread
    over the logarithm below it, as requests of mixed age have them."""
    rng = random.Random(c["ctx"] * 1000003 + c["batch"])
    return [c["ctx"]] + [max(1, int(c["ctx"] * math.exp(-2.0 * rng.random()))) for _ in range(c["batch"] - 1)]


def work(c) -> dict:
    planes = 2 * c["layers"]
    slot = c["heads"] * c["dim"] * 2
    if c["kind"] == "migrate":
        n = _blocks(c, c["tokens"] + c["batches"] * c["append"])
        return {"bytes": planes * (2 * n * _tile(c) + 2 * c["batches"] * c["append"] * slot), "flops": 0}
    if c["kind"] == "finish":
        return {"bytes": planes * 2 * _blocks(c, c["tokens"]) * _tile(c), "flops": 0}
    if c["kind"] == "stage":
        return {"bytes": planes * 2 * c["pairs"] * _tile(c), "flops": 0}
    if c["kind"] in ("fuse", "host"):     # out of the pool, into staging and out of it, into the pool
        return {"bytes": planes * 4 * c["pairs"] * _tile(c), "flops": 0}
    if c["kind"] == "write":
        return {"bytes": planes * 2 * c["requests"] * c["tokens"] * slot, "flops": 0}
    lens = _context_lengths(c)
    rows = c["layers"] * c["batch"] * c["heads"] * c["group"] * c["dim"]
    n = sum(lens) * planes * slot + rows * 6
    if c["call"] == "carry":
        n += c["ctx"] // c["block"] * planes * _tile(c)
    return {"bytes": n, "flops": 4 * sum(lens) * c["layers"] * c["heads"] * c["group"] * c["dim"]}


def tolerance(c):
    """Copies and writes: the bytes themselves.  Attention: fp32 sums of
    products of 16-bit inputs, in any order."""
    if c["kind"] != "decode":
        return "exact"
    return {"rel": 1e-5, "max": 4e-4}


# ---- inputs -------------------------------------------------------------------

def _fill(t, gen, step=1 << 28):
    flat = t.view(-1)
    for at in range(0, flat.numel(), step):
        flat[at:at + step].normal_(generator=gen)


def _pool(c, blocks, gen, layouts=("NHD", "NHD"), fill=True):
    """A pool of ``blocks`` blocks whose layer tensors are slices of one
    tensor: (handle, tensor [2][layers][blocks][block][heads][dim])."""
    t = torch.empty((2, c["layers"], blocks, c["block"], c["heads"], c["dim"]), dtype=DTYPES[c["dtype"]],
                    device="cuda")
    if fill:
        _fill(t, gen)
    else:
        t.zero_()
    pool = llmig.Pool(list(t[0].unbind(0)), list(t[1].unbind(0)), tuple(LAYOUTS[x] for x in layouts))
    return pool, t


def _pool_blocks(n):
    """Blocks of a pool in which ``n`` belong to the requests at hand and a
    quarter as many to others."""
    return n + n // 4 + 3


_streams: list = []


def _two_streams():
    """The migration and the decode stream of a program, taken once."""
    if not _streams:
        _streams.extend(harness.concurrent_streams(2)[0])
    return _streams


def prepare(c, seed: int) -> dict:
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    kind = c["kind"]
    s = {"case": c}
    if kind in ("migrate", "finish"):
        total = c["tokens"] + c.get("batches", 0) * c.get("append", 0)
        need = _blocks(c, total)
        nb = _pool_blocks(need)
        s["src"], _ = _pool(c, nb, gen)
        s["dst"], s["out"] = _pool(c, nb, gen, fill=False)
        s["table"] = rng.permutation(nb).astype(np.int32)[:need]
        s["free"] = rng.permutation(nb).astype(np.int32)
        if kind == "migrate":
            s["streams"] = _two_streams()
            s["appends"] = []
            for _ in range(c["batches"]):
                a = torch.empty((c["layers"], 2, c["append"], c["heads"] * c["dim"]), dtype=DTYPES[c["dtype"]],
                                device="cuda")
                _fill(a, gen)
                s["appends"].append(a.view(torch.uint8))
    elif kind in ("stage", "fuse", "host"):
        nb = _pool_blocks(c["pairs"])
        ends = [x.split("/") for x in c.get("layouts", "NHD/NHD>NHD/NHD").split(">")]
        s["src"], _ = _pool(c, nb, gen, ends[0])
        s["dst"], s["out"] = _pool(c, nb, gen, ends[1], fill=False)
        s["from"] = rng.permutation(nb).astype(np.int32)[:c["pairs"]]
        s["to"] = rng.permutation(nb).astype(np.int32)[:c["pairs"]]
        if c.get("ids") == "device":
            s["from"], s["to"] = torch.from_numpy(s["from"]).cuda(), torch.from_numpy(s["to"]).cuda()
        nbytes = c["layers"] * 2 * _tile(c)
        if kind == "fuse":
            s["staging"] = torch.empty(c["pairs"] * nbytes // 2, dtype=torch.int16, device="cuda")
            s["staged"] = tuple(LAYOUTS[x] for x in ends[0])
        if kind == "host":
            s["bufs"] = [torch.empty(c["chunk"] * nbytes, dtype=torch.uint8, pin_memory=True) for _ in range(2)]
            s["streams"] = _two_streams()
    elif kind == "decode":
        lens = _context_lengths(c)
        per = [_blocks(c, n) for n in lens]
        nb = _pool_blocks(sum(per))
        s["pool"], s["kv"] = _pool(c, nb, gen)
        order = rng.permutation(nb).astype(np.int32)
        tables = np.zeros((c["batch"], max(per)), np.int32)
        at = 0
        for b, n in enumerate(per):
            tables[b, :n] = order[at:at + n]
            at += n
        s["tables"], s["lens"] = torch.from_numpy(tables).cuda(), lens
        shape = (c["layers"], c["batch"], c["heads"] * c["group"], c["dim"])
        s["q"] = torch.empty(shape, dtype=DTYPES[c["dtype"]], device="cuda")
        _fill(s["q"], gen)
        s["scale"] = 1.0 / math.sqrt(c["dim"])
        s["attn"] = torch.empty(shape, dtype=torch.float32, device="cuda")
        if c["call"] != "noalloc":
            n = llmig.decode_workspace_bytes(lens, c["layers"], shape[2], c["dim"])
            s["ws"] = torch.empty(max(16, n), dtype=torch.uint8, device="cuda")
        if c["call"] == "carry":
            whole = c["ctx"] // c["block"]
            n = _pool_blocks(whole)
            s["dst"], s["out"] = _pool(c, n, gen, fill=False)
            s["to"] = torch.from_numpy(rng.permutation(n).astype(np.int32)[:whole]).cuda()
    else:
        need = _blocks(c, c["first"] + c["tokens"])
        nb = _pool_blocks(need * c["requests"])
        s["pool"], s["out"] = _pool(c, nb, gen, c["layouts"].split("/"), fill=False)
        order = rng.permutation(nb).astype(np.int32)
        s["tables"] = [order[k * need:(k + 1) * need].copy() for k in range(c["requests"])]
        s["data"] = []
        for _ in range(c["requests"]):
            a = torch.empty((c["layers"], 2, c["tokens"], c["heads"] * c["dim"]), dtype=DTYPES[c["dtype"]],
                            device="cuda")
            _fill(a, gen)
            s["data"].append(a)
    return s


# ---- one pass ------------------------------------------------------------------

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "migrate":
        m, _ = migrate.run_scheduled(s["src"], s["dst"], s["table"], s["free"], c["tokens"], s["appends"], *s["streams"])
        return {"dst": s["out"].view(torch.int16), "table": m.commit()}
    if kind == "finish":
        m = migrate.Migration(s["src"], s["dst"], s["table"], s["free"], torch.cuda.current_stream())
        m.finish(c["tokens"])
        return {"dst": s["out"].view(torch.int16), "table": m.commit()}
    if kind == "stage":
        llmig.llmig_stage(s["src"], s["dst"], s["from"], s["to"])
        return {"dst": s["out"].view(torch.int16)}
    if kind == "fuse":
        llmig.llmig_pack(s["src"], s["from"], s["staging"])
        llmig.llmig_unpack_layout(s["dst"], s["to"], s["staging"], s["staged"])
        return {"dst": s["out"].view(torch.int16), "staging": s["staging"]}
    if kind == "host":
        pack, unpack = s["streams"]
        here = torch.cuda.current_stream()
        pack.wait_stream(here)
        pack.wait_stream(unpack)         # the buffers' last readers
        migrate.run_host_staged(s["src"], s["dst"], s["from"], s["to"], s["bufs"], pack, unpack, c["chunk"])
        here.wait_stream(unpack)
        return {"dst": s["out"].view(torch.int16)}
    if kind == "write":
        for table, data in zip(s["tables"], s["data"]):
            llmig.llmig_write_tokens(s["pool"], table, c["first"], data)
        return {"pool": s["out"].view(torch.int16)}
    args = (s["pool"], s["q"], s["tables"], s["lens"], s["scale"])
    if c["call"] == "noalloc":
        llmig.llmig_decode_attention_noalloc(*args, s["attn"])
        return {"out": s["attn"]}
    if c["call"] == "workspace" or not s["to"].numel():
        llmig.llmig_decode_attention(*args, s["ws"], s["attn"])
        return {"out": s["attn"]}
    llmig.llmig_decode_attention_migrate(*args, s["ws"], s["attn"], s["dst"], 0, s["to"], 0)
    return {"out": s["attn"], "dst": s["out"].view(torch.int16)}


def exact(c, seed: int):
    """Decode attention in float64; the other kinds compute no numbers."""
    if c["kind"] != "decode":
        return None
    s = prepare(c, seed)
    heads, dim, group = c["heads"], c["dim"], c["group"]
    out = torch.zeros(s["attn"].shape, dtype=torch.float64, device="cuda")
    for b, n in enumerate(s["lens"]):
        ids = s["tables"][b, :_blocks(c, n)].long()
        for layer in range(c["layers"]):
            k, v = (s["kv"][j, layer][ids].reshape(-1, heads, dim)[:n].double().transpose(0, 1).contiguous()
                    for j in (0, 1))
            q = s["q"][layer, b].double().reshape(heads, group, dim)
            p = torch.softmax(torch.matmul(q, k.transpose(1, 2).contiguous()) * s["scale"], dim=-1)
            out[layer, b] = torch.matmul(p, v).reshape(heads * group, dim)
    if c["call"] == "carry" and s["to"].numel():
        return {"out": out, "dst": None}
    return {"out": out}

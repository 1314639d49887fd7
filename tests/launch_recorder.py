"""Runs library calls over a stand-in HIP runtime (fake_hip.c) and prints what
they launch, as JSON.  A process of its own, without torch:

    python launch_recorder.py FAKE_HIP.so LIBLLMIG.so < calls.json

A call is a dict: ``call`` and its arguments as below.  For each: {"rc",
"launches": [{"kernel", "grid", "block", "lds", ...fields of its arguments}]}."""
import ctypes
import json
import sys

import numpy as np

U32, I32, U64, P = ctypes.c_uint32, ctypes.c_int32, ctypes.c_uint64, ctypes.c_uint64
INLINE, MAX_BATCH = 256, 256


class Divisor(ctypes.Structure):
    _fields_ = [("d", U32), ("m", U32), ("shift", U32)]


# The kernels' argument structures, as the sources declare them.
class CopyArgs(ctypes.Structure):
    _fields_ = [("src_tab", P), ("dst_tab", P), ("src_lin", P), ("dst_lin", P), ("src_ids_dev", P),
                ("dst_ids_dev", P), ("tile_bytes", U32), ("num_layers", U32), ("planes", U32), ("pairs", U32),
                ("spans_per_tile", U32), ("items", U32), ("first_item", U32), ("by_span", Divisor),
                ("by_pair", Divisor), ("xcd_runs", U32), ("lin_first", U32), ("lin_pairs", U32),
                ("ids", U32 * (2 * INLINE))]


class ConvertArgs(ctypes.Structure):
    _fields_ = [("src_tab", P), ("dst_tab", P), ("src_lin", P), ("src_ids_dev", P), ("dst_ids_dev", P),
                ("magic_row", U64), ("magic_bs", U64), ("magic_t", U64), ("tile_bytes", U32), ("num_layers", U32),
                ("heads", U32), ("block_size", U32), ("row_chunks", U32), ("t_chunks", U32), ("chunks", U32),
                ("pairs", U32), ("units", U32), ("first_unit", U32), ("by_head", Divisor), ("by_pair", Divisor),
                ("lin_first", U32), ("lin_pairs", U32), ("first_slot", U32), ("tokens", U32), ("layouts", I32 * 4),
                ("ids", U32 * (2 * INLINE))]


class AttnArgs(ctypes.Structure):
    _fields_ = [("k_tab", P), ("q", P), ("tables", P), ("ws", P), ("out", P), ("scale", ctypes.c_float),
                ("num_layers", U32), ("batch", U32), ("q_heads", U32), ("kv_heads", U32), ("block_size", U32),
                ("table_stride", U32), ("item_base", U32), ("layer_items", U32), ("n_records", U32), ("part_tokens", U32),
                ("item_end", U32 * MAX_BATCH), ("ctx", I32 * MAX_BATCH), ("seq", U32 * (MAX_BATCH // 2)),
                ("dst_tab", P), ("mig_ids", P), ("mig_seq", I32), ("mig_from", I32), ("mig_to", I32),
                ("dst_layer_bytes", U32), ("dst_blocks", I32)]


class AttnReduceArgs(ctypes.Structure):
    _fields_ = [("ws", P), ("out", P), ("num_layers", U32), ("batch", U32), ("q_heads", U32), ("head_dim", U32),
                ("n_records", U32), ("row_base", U64), ("seqs", U32), ("seq_end", U32 * MAX_BATCH),
                ("seq", ctypes.c_uint8 * MAX_BATCH)]


class WriteArgs(ctypes.Structure):
    _fields_ = [("tab", P), ("data", P), ("slot_bytes", U32), ("tile_bytes", U32), ("block_size", U32),
                ("num_layers", U32), ("head_dim", U32), ("row_chunks", U32), ("layouts", I32 * 2),
                ("data_tokens", U32), ("first_token", U32), ("tokens", U32), ("first_slot", U32), ("blocks", U32),
                ("rows_per_run", U32), ("first_item", U32), ("by_row", Divisor), ("by_block", Divisor),
                ("ids", I32 * INLINE)]


STRUCTS = {"write_rows": WriteArgs, "write_token_slots": WriteArgs, "attn_partial_mfma": AttnArgs, "attn_reduce": AttnReduceArgs, "copy_rows": CopyArgs, "copy_tiles": CopyArgs, "convert_slabs": ConvertArgs, "convert_tiles": ConvertArgs}


class Desc(ctypes.Structure):
    _fields_ = [(n, I32) for n in ("num_layers", "num_blocks", "block_size", "num_kv_heads", "head_dim", "elem_bytes")] \
        + [("k_ptrs", ctypes.POINTER(U64)), ("v_ptrs", ctypes.POINTER(U64)), ("k_layout", I32), ("v_layout", I32)]


class SlabWriteArgs(ctypes.Structure):
    _fields_ = ConvertArgs._fields_[:-1] + [("ids", U32 * INLINE)]


STRUCTS["write_slabs"] = SlabWriteArgs

HOST_MEMORY = 1 << 46
launches = []


def fields(args):
    out = {}
    for name, kind in args._fields_:
        v = getattr(args, name)
        if isinstance(v, ctypes.Array):
            v = list(v)
        elif isinstance(v, ctypes.Structure):
            continue
        out[name] = v
    return out


@ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.POINTER(U32), U64, ctypes.c_void_p)
def on_launch(name, gb, lds, args):
    name = name.decode()
    rec = {"kernel": name, "grid": gb[0], "block": gb[3], "lds": lds}
    for key, struct in STRUCTS.items():
        if key in name:
            rec["kernel"] = key
            rec["template"] = [int(x) for x in __import__("re").findall(r"Li(\d+)E", name)]
            rec.update(fields(struct.from_address(args)))
    launches.append(rec)


fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.fake_hip_on_launch(on_launch)
lib = ctypes.CDLL(sys.argv[2])
pools = {}


def pool(layers, blocks, bs, heads, dim, layouts=(0, 0), at=1):
    key = (layers, blocks, bs, heads, dim, tuple(layouts), at)
    if key not in pools:
        size = blocks * bs * heads * dim * 2
        ptr = [(at << 43) + i * (size + 256) // 256 * 256 for i in range(2 * layers)]
        k, v = (U64 * layers)(*ptr[:layers]), (U64 * layers)(*ptr[layers:])
        desc = Desc(layers, blocks, bs, heads, dim, 2, k, v, *layouts)
        h = ctypes.c_void_p()
        assert lib.llmig_pool_create(ctypes.byref(desc), ctypes.byref(h)) == 0
        pools[key] = h
    return pools[key]


def ids(values):
    a = np.asarray(values, np.int32)
    return a, a.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(a.size)


def stage(pool_args, src, dst, layouts=((0, 0), (0, 0))):
    a, pa, n = ids(src)
    b, pb, _ = ids(dst)
    return lib.llmig_stage(pool(*pool_args, layouts[0], 1), pool(*pool_args, layouts[1], 2), pa, pb, n, 0, None)


def fuse(call, pool_args, blocks, staging, layouts=(0, 0), staging_layouts=(0, 0)):
    a, pa, n = ids(blocks)
    where = ctypes.c_void_p(HOST_MEMORY if staging == "host" else 1 << 30)
    size = ctypes.c_int64(1 << 45)
    p = pool(*pool_args, layouts, 1)
    if call == "unpack_layout":
        return lib.llmig_unpack_layout(p, pa, n, 0, where, size, *staging_layouts, None)
    return getattr(lib, "llmig_" + call)(p, pa, n, 0, where, size, None)


def decode(pool_args, ctx, group, workspace="full", carry=None, seq=0):
    """workspace: "full" (the size the library returns), "least" (2048 tokens a
    partition), "none" (llmig_decode_attention_noalloc).  carry: blocks of
    sequence `seq` that the call carries into another pool."""
    layers, _, bs, heads, dim = pool_args
    c, pc, _ = ids(ctx)
    q_heads, stride = heads * group, max(1, max(-(-n // bs) for n in ctx))
    size = ctypes.c_int64()
    assert lib.llmig_decode_attention_workspace(pc, len(ctx), layers, q_heads, dim, ctypes.byref(size)) == 0
    least = layers * q_heads * (dim + 4) * 4 * sum(-(-n // 2048) for n in ctx)
    assert size.value >= least
    q, tables, out, ws = (ctypes.c_void_p(a << 44) for a in (1, 2, 3, 4))
    scale = ctypes.c_float(0.1)
    if workspace == "none":
        return lib.llmig_decode_attention_noalloc(pool(*pool_args), 0, q, len(ctx), q_heads, tables, stride, pc,
                                                  scale, out, None)
    if carry:
        return lib.llmig_decode_attention_migrate(
            pool(*pool_args), 0, q, len(ctx), q_heads, tables, stride, pc, scale, ws, size, out,
            pool(*pool_args, (0, 0), 2), seq, ctypes.c_void_p(5 << 44), ctypes.c_int64(0), ctypes.c_int64(carry), None)
    return lib.llmig_decode_attention(pool(*pool_args), 0, q, len(ctx), q_heads, tables, stride, pc, scale, ws,
                                      ctypes.c_int64(size.value if workspace == "full" else least), out, None)


def write(pool_args, table, first, tokens, layouts=(0, 0)):
    t, pt, n = ids(table)
    return lib.llmig_write_tokens(pool(*pool_args, layouts), pt, n, ctypes.c_int64(first), ctypes.c_int64(tokens),
                                  ctypes.c_void_p(1 << 30), None)


CALLS = {"stage": stage, "decode": decode, "write": write}


def main():
    out = []
    for c in json.load(sys.stdin):
        launches.clear()
        kind = c.pop("call")
        rc = CALLS[kind](**c) if kind in CALLS else fuse(kind, **c)
        out.append({"rc": rc, "launches": list(launches)})
    json.dump(out, sys.stdout)


main()

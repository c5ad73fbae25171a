"""Timed cases of the KV pool: what a serving engine has the library do, through its public calls.

A case fixes a KV shape (layers, KV heads, head_dim, tokens per block, bytes per element), the pool's
chunk layout and regions, one call pattern, and the number of blocks.  Two kinds of pool are in use:

* ``configured``: weights 4:4:1:1:1:1 over two host regions and four HBM staging regions, the ratios
  of the paper's DRAM and SSDs.  Two thirds of a request cross the host link.
* ``measured``: Eq. 1 with the bandwidths that a pool created without weights measures on an MI355X
  (MB/s, written down here so that every run places alike).  Nearly every block lies in HBM.

The library copies bytes and computes no numbers, so results are compared bit for bit, and there is
no value of higher precision to compare them with.  Outputs are whole buffers (the engine cache after
a retrieve, the written ranges of the pool after a store) seen as 64-bit words.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_14779_amd import kvpool as K

SECTOR = 4096
KINDS = ("host", "host", "staging", "staging", "staging", "staging")
WEIGHTS = {"configured": (4, 4, 1, 1, 1, 1),
           "measured": (28700, 28700, 2850000, 2850000, 2850000, 2850000)}
BIGGEST = 8192 * 2 * 32 * 8 * 16 * 128 * 2     # bytes of the largest request: 128K LLaMA-shaped tokens
LINK_MOST = 512 * 2 * 32 * 8 * 16 * 128 * 2    # and of the largest one on the configured pool


def _case(op, layers, heads, head_dim, blocks, *, block=16, elem=2, layout=0, pool="measured", table="permuted",
          name=None):
    c = {"op": op, "layers": layers, "heads": heads, "head_dim": head_dim, "block": block, "elem": elem,
         "layout": layout, "pool": pool, "blocks": blocks, "table": table}
    return dict(c, name=name) if name else c


def listed():
    return [
        # every decoding step that fills a block offloads it: one 2 MiB block over the host link
        _case("extend_store", 32, 8, 128, 1, pool="configured", name="decode step, 1 block"),
        # a short shared prefix (256 tokens of LLaMA-8B) comes back before a prefill
        _case("retrieve", 32, 8, 128, 16, pool="configured", name="prefix of 16 blocks"),
        # the same with the KV heads of LLaMA-8B split over 8 GPUs: 4 KiB chunks, 2K tokens, from HBM
        _case("retrieve", 32, 1, 128, 128, name="prefix of 128, 1 head"),
        # long contexts from HBM staging, the three models' shapes; LLaMA's is the headline request
        _case("retrieve", 24, 8, 64, 8192, name="gpt-oss 128K"),
        _case("retrieve", 32, 8, 128, 8192, table="fragmented", name="llama 128K"),
        # the offload of a long context after its prefill
        _case("store", 48, 4, 128, 4096, name="qwen3 64K store"),
        # continuous batching: four requests of different lengths, part of each absent, one call
        _case("batch", 48, 4, 128, 3271, name="qwen3 batch of 4"),
        # a pool that keeps chunks token by token, as the engine's prefill writes them
        _case("retrieve", 32, 8, 128, 2048, layout=1, table="fragmented", name="llama 32K token-major"),
        # one turn of a chat: the context is placed, offloaded, fetched again and released
        _case("turn", 24, 8, 64, 1024, layout=1, name="gpt-oss 16K turn"),
        # layer by layer, for an engine that starts on layer 0 while the rest is fetched
        _case("layers", 32, 8, 128, 2048, table="fragmented", name="llama 32K layerwise"),
        # a context striped over both kinds of region, where the host link sets the time
        _case("retrieve", 32, 8, 128, 512, pool="configured", table="fragmented", name="llama 8K, host link"),
        # 8-bit KV of an odd shape, by the call that allocates nothing
        _case("noalloc", 20, 5, 80, 1000, elem=1, name="8-bit odd shape, noalloc"),
    ]


def draw(rng):
    while True:
        op = rng.choice(("retrieve", "retrieve", "retrieve", "store", "store", "extend_store", "batch", "turn", "layers",
                         "noalloc", "copy_engines"))
        shape = rng.choice(((32, 8, 128), (24, 8, 64), (48, 4, 128), (32, 1, 128), None))
        layers, heads, head_dim = shape or (rng.randint(8, 48), rng.choice((1, 2, 3, 4, 5, 6, 8)),
                                            rng.choice((64, 80, 96, 112, 128)))
        elem = rng.choice((2, 2, 2, 1, 4))
        block = rng.choice((16, 16, 16, 8, 32))
        pool = "configured" if op == "copy_engines" else rng.choice(("measured", "measured", "configured"))
        block_bytes = 2 * layers * heads * block * head_dim * elem
        most = (LINK_MOST if pool == "configured" else BIGGEST) // (2 if op == "turn" else 1) // block_bytes
        blocks = int(round(math.exp(rng.uniform(0, math.log(32 if op == "extend_store" else 8192)))))
        if blocks <= most and blocks * block_bytes >= 1 << 19:
            return _case(op, layers, heads, head_dim, blocks, block=block, elem=elem, layout=rng.choice((0, 0, 1)),
                         pool=pool, table=rng.choice(("permuted", "fragmented")))


class _RegionWords:
    """The 64-bit words of one range of a region where they lie; keeps its pool open."""

    def __init__(self, pool, region, offset, nbytes):
        info = pool.region_info(region)
        self.pool = pool
        host = info["type"] == K.REGION_HOST
        at = (info["host_ptr"] if host else info["device_ptr"]) + offset
        view = {"shape": (nbytes // 8,), "typestr": "<i8", "data": (at, False), "strides": None, "version": 2}
        if host:
            self.__array_interface__ = dict(view, version=3)
        else:
            self.__cuda_array_interface__ = view

    def tensor(self):
        if hasattr(self, "__array_interface__"):
            return torch.from_numpy(np.asarray(self))
        return torch.as_tensor(self, device="cuda")


def _written(pool, loc_map, block_bytes):
    out = []
    for r in range(len(KINDS)):
        off = loc_map["offset"][loc_map["region"] == r]
        if len(off):
            lo = int(off.min())
            out.append(_RegionWords(pool, r, lo, int(off.max()) + block_bytes - lo).tensor())
    return out


def _cache(case, slots, gen=None):
    """Engine cache [layers][K/V][slots][heads][tokens][head_dim]; with a generator its values: N(0, 1), or any
    bytes where the elements are quantised to 8 bits."""
    shape = (case["layers"], 2, slots, case["heads"], case["block"], case["head_dim"])
    dtype = {1: torch.int8, 2: torch.bfloat16, 4: torch.float32}[case["elem"]]
    if gen is None:
        return torch.zeros(shape, dtype=dtype, device="cuda")
    t = torch.empty(shape, dtype=dtype, device="cuda")
    for layer in t:
        if case["elem"] == 1:
            layer.random_(-128, 128, generator=gen)
        else:
            layer.normal_(generator=gen)
    return t


def _pointers(cache):
    return [c[0].data_ptr() for c in cache], [c[1].data_ptr() for c in cache]


def _slots(case, n, rng):
    """n slots of a cache that is a fifth in use: ascending, or in any order."""
    total = n + n // 4 + 1
    free = rng.permutation(total)[:n]
    return total, (np.sort(free) if case["table"] == "fragmented" else free).astype(np.int32)


def _requests(case, rng):
    """(blocks of the context, blocks of it in the pool) of every request."""
    n = case["blocks"]
    if case["op"] != "batch":
        return [(n, n)]
    cut = np.sort(rng.choice(np.arange(1, n), size=3, replace=False)) if n >= 8 else np.arange(1, min(n, 4))
    present = np.diff(np.concatenate([[0], cut, [n]]))
    return [(int(p) + int(rng.integers(0, p + 1)), int(p)) for p in present]


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    spec = K.KVSpec(case["layers"], case["heads"], case["head_dim"], case["block"], case["elem"], case["layout"])
    weights, op, n = WEIGHTS[case["pool"]], case["op"], case["blocks"]
    reqs = _requests(case, rng)
    sets = [p for _, p in reqs] + ([8] if op == "extend_store" else [])   # 8: the context before this step
    room = [sum(-(-(w * s // sum(weights) + 1) * spec.block_bytes // SECTOR) * SECTOR for s in sets) for w in weights]
    pool = K.KVPool([K.Region(kind, size) for kind, size in zip(KINDS, room)], weights, spec)
    if op == "copy_engines":
        pool.set_launch(K.CLASS_HOST, K.OP_RETRIEVE, 0, K.LAUNCH_SDMA)
    src_slots, src_table = _slots(case, n, rng)
    src = _cache(case, src_slots, gen)
    state = {"op": op, "pool": pool, "spec": spec, "n": n, "layers": case["layers"]}
    if op in ("store", "extend_store"):
        if op == "store":
            loc_map = pool.place(1, n)
        else:
            pool.place(1, 8)
            loc_map = pool.extend(1, n)
        state.update(map=loc_map, table=src_table, slots=src_slots, keep=src, out=_written(pool, loc_map, spec.block_bytes))
        state["k"], state["v"] = _pointers(src)
        return state
    dst_slots, dst_table = _slots(case, n, rng)
    dst = _cache(case, dst_slots)
    state.update(slots=dst_slots, table=dst_table, out=[dst.view(-1).view(torch.int64)])
    state["k"], state["v"] = _pointers(dst)
    src_k, src_v = _pointers(src)
    if op == "turn":
        state.update(keep=src, src_slots=src_slots, src_table=src_table, src_k=src_k, src_v=src_v)
        return state
    stream = torch.cuda.current_stream().cuda_stream
    maps, tables, at = [], [], 0
    for i, (context, present) in enumerate(reqs):
        loc_map = pool.place(i + 1, present)
        pool.store(loc_map, src_table[at:at + present], src_slots, src_k, src_v, stream)
        whole = np.zeros(context, dtype=K.LOC_DTYPE)
        whole[:present] = loc_map
        whole["region"][present:] = K.ABSENT
        maps.append(whole)
        tables.append(np.concatenate([dst_table[at:at + present], np.full(context - present, -1, np.int32)]))
        at += present
    state.update(map=np.concatenate(maps), table=np.concatenate(tables))
    torch.cuda.synchronize()   # the source cache is given back here
    return state


def run(state):
    pool, table, slots, k, v = state["pool"], state["table"], state["slots"], state["k"], state["v"]
    stream = torch.cuda.current_stream().cuda_stream
    op = state["op"]
    if op in ("retrieve", "copy_engines"):
        pool.retrieve_request(1, table, slots, k, v, stream)
    elif op in ("store", "extend_store"):
        pool.store(state["map"], table, slots, k, v, stream)
    elif op == "batch":
        pool.retrieve(state["map"], table, slots, k, v, stream)
    elif op == "noalloc":
        pool.retrieve_noalloc(state["map"], table, slots, k, v, stream)
    elif op == "layers":
        for layer in range(state["layers"]):
            pool.retrieve_layers(state["map"], table, slots, layer, layer + 1, k, v, stream)
    else:   # "turn"
        loc_map = pool.place(1, state["n"])
        pool.store(loc_map, state["src_table"], state["src_slots"], state["src_k"], state["src_v"], stream)
        pool.retrieve_request(1, table, slots, k, v, stream)
        pool.release(1)
    return state["out"]


def work(case):
    moved = 2 * case["layers"] * case["heads"] * case["block"] * case["head_dim"] * case["elem"] * case["blocks"]
    return {"bytes": 2 * moved * (2 if case["op"] == "turn" else 1), "flops": 0}   # each byte read once and written once


def tolerance(case):
    return "exact"

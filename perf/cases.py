"""The work users of this engine give it, as cases that can be timed and compared.

A case names the shape of a paged KV cache (layers, KV heads, head dimension,
tokens per block, bytes per element), the call (`kind`) and its lists.  Every
kind goes through the public entry points of the Python binding, waits the way
a caller waits, and returns the whole cache and the whole pool (the reader: its
checksum).  Shapes are those of the workloads module, their shards under tensor
parallelism (fewer KV heads per GPU), and generic ones that are a power of two
nowhere.
"""
import math

import numpy as np
import torch

from paper_2601_20309_amd import binding as B
from paper_2601_20309_amd import workloads as W

MiB = 1 << 20


def _case(kind, layers, heads, dim, tokens, elem, n_out, n_in, **opt):
    c = dict(kind=kind, layers=layers, heads=heads, dim=dim, tokens=tokens, elem=elem, n_out=n_out, n_in=n_in,
             host_layout="block_first", hbm_layout="layer_first", path="auto", chunk_layers=0, slots="scattered")
    c.update(opt)
    return c


def listed():
    llama, long70b, qwen = (32, 8, 128, 16, 2), (80, 8, 128, 32, 2), (64, 8, 128, 16, 2)
    llama_tp8, long70b_tp8 = (32, 1, 128, 16, 2), (80, 1, 128, 32, 2)
    named = {
        # the smallest rotation there is a configuration for: 8 blocks of 16 KiB each way, all latency
        "tiny_rotate": _case("rotate", 2, 2, 64, 16, 2, 8, 8),
        # the entry point that allocates nothing, with the few blocks a decode iteration swaps
        "static_few_blocks": _case("static", *llama, 4, 3),
        # the eager step of one iteration of the serving loop: 45 filled blocks to DRAM, beside execution
        "eager_step_out": _case("swap_out", *llama, 45, 0),
        # the headline: one 2048-token request out, another in (bench.py's workload)
        "rotate_2048_tokens": _case("rotate", *llama, 128, 128),
        # the largest: 4096 tokens each way of the 64-layer shape, 1 GiB per direction
        "rotate_1gib_each_way": _case("rotate", *qwen, 256, 256),
        # two iterations of the block table: a request leaves, one comes back, the eager copies of a third ride along
        "serve_two_iterations": _case("serve", *llama, 24, 61),
        # resuming a long request layer by layer, so that the model can start on the first layers
        "resume_layered_70b": _case("swap_in", *long70b, 0, 37, chunk_layers=4),
        # one of eight tensor-parallel shards, pool laid out like the cache: segments of 8 KiB
        "shard_layer_first": _case("rotate", *long70b_tp8, 97, 83, host_layout="layer_first"),
        # segments of 1200 bytes, which no tile divides
        "ragged_rotate": _case("rotate", 24, 3, 40, 5, 2, 701, 633),
        # the path that takes least from the model running beside it: pack, DMA engines, unpack
        "staged_rotate": _case("rotate", *llama, 120, 96, path="sdma_staged"),
        # decode over everything resident: 8 GiB of KV read once
        "reader_8gib": _case("reader", *llama, 4096, 0),
        # the same on one of eight shards: 1500 blocks in segments of 4 KiB
        "reader_shard": _case("reader", *llama_tp8, 1500, 0),
    }
    return [dict(c, name=n) for n, c in named.items()]


def draw(rng):
    pick = rng.choice
    logu = lambda lo, hi: math.exp(rng.uniform(math.log(lo), math.log(hi)))  # noqa: E731
    kind = pick(["rotate"] * 8 + ["swap_out", "swap_out", "swap_in", "swap_in", "static", "static", "serve", "serve"]
                + ["reader"] * 4)
    if rng.random() < 0.5:
        layers, heads, dim, tokens = pick([(32, 8, 128, 16), (80, 8, 128, 32), (64, 8, 128, 16), (32, 1, 128, 16),
                                           (80, 1, 128, 32), (32, 2, 128, 16), (2, 2, 64, 16), (4, 8, 128, 16)])
        elem = pick([2, 2, 2, 1])
    else:
        layers, heads = round(logu(2, 80)), pick([1, 2, 3, 4, 5, 8])
        dim, tokens, elem = pick([40, 64, 80, 96, 128]), pick([5, 7, 8, 16, 16, 32]), pick([2, 2, 2, 1, 4])
    if kind == "reader" and (heads * dim * tokens * elem) % 16:
        tokens = 16                 # the reader takes whole 16-byte vectors
    block = 2 * layers * heads * dim * tokens * elem
    opt = dict(host_layout=pick(["block_first", "block_first", "layer_first"]),
               hbm_layout=pick(["layer_first", "layer_first", "layer_first", "block_first"]))
    if kind == "reader":
        n = max(1, min(6000, round(logu(1 * MiB, 4096 * MiB) / block)))
        return _case(kind, layers, heads, dim, tokens, elem, n, 0, **opt)
    if kind == "rotate":
        opt["path"] = pick(["auto"] * 7 + ["zerocopy", "sdma_staged", "sdma_staged"])
        opt["chunk_layers"] = pick([0, 0, 0, max(1, layers // 8)])
        opt["slots"] = pick(["scattered", "scattered", "runs"])
    most = 512 * MiB
    if opt.get("path") == "sdma_staged" and opt["host_layout"] == "layer_first" and opt["slots"] == "scattered":
        most = 16 * MiB             # one DMA copy per segment: keep the pass short
    total = logu(64 << 10, most)
    n_out = max(1, min(2500, round(total / block * rng.uniform(0.4, 1.0))))
    n_in = max(1, min(2500, round(total / block * rng.uniform(0.2, 1.0))))
    if kind == "swap_out":
        n_in = 0
    if kind == "swap_in":
        n_out = 0
        opt["chunk_layers"] = pick([0, 0, max(1, layers // 8)])
    return _case(kind, layers, heads, dim, tokens, elem, n_out, n_in, **opt)


def _seg(case):
    return case["heads"] * case["dim"] * case["tokens"] * case["elem"]


def _block(case):
    return 2 * case["layers"] * _seg(case)


def _sizes(case):
    """Blocks of the cache and slots of the pool: room to be scattered in."""
    if case["kind"] == "reader":
        return case["n_out"] + case["n_out"] // 2 + 16, 8
    if case["kind"] == "serve":     # two rotating requests of n_in blocks, one growing of n_out
        n = case["n_out"] + 2 * case["n_in"]
        return n + 8, n + 8
    n = case["n_out"] + case["n_in"]
    return 2 * n + 16, n + n // 4 + 8


def _values(n_bytes, elem, g):
    """KV values N(0, 1) of the element type, as bytes on the GPU."""
    if elem == 4:
        return torch.empty(n_bytes // 4, dtype=torch.float32, device="cuda").normal_(generator=g).view(torch.uint8)
    v = torch.empty(n_bytes // min(elem, 2), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    return (v if elem == 2 else v.to(torch.float8_e4m3fn)).view(torch.uint8)


def _words(t, case):
    """The same memory in the widest whole numbers that divide a segment."""
    for size, dtype in ((8, torch.int64), (4, torch.int32), (2, torch.int16)):
        if _seg(case) % size == 0:
            return t.view(dtype)
    return t


def _inputs(case, seed):
    """(cache on the GPU, pool bytes on the GPU, out ids, out slots, in ids, in slots)"""
    g = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    nb, ns = _sizes(case)
    cache = _values(nb * _block(case), case["elem"], g)
    pool = _values(ns * _block(case), case["elem"], g)
    n_out, n_in = (case["n_out"], case["n_in"]) if case["kind"] != "serve" else (0, 0)
    ids = rng.permutation(nb)[:n_out + n_in].astype(np.int32)
    if case["kind"] == "reader":
        slots = np.zeros(0, np.int32)
    elif case["slots"] == "runs":
        slots = (np.arange(n_out + n_in) + int(rng.integers(0, ns - n_out - n_in + 1))).astype(np.int32)
    else:
        slots = rng.permutation(ns)[:n_out + n_in].astype(np.int32)
    return cache, pool, ids[:n_out], slots[:n_out], ids[n_out:], slots[n_out:]


def prepare(case, seed):
    cache, pool, oi, os_, ii, is_ = _inputs(case, seed)
    nb, ns = _sizes(case)
    shape = W.KVShape(case["layers"], case["heads"], case["dim"], case["tokens"], nb, ns, case["elem"])
    cfg = B.make_config(
        shape, B.KV_HOST_BLOCK_FIRST if case["host_layout"] == "block_first" else B.KV_HOST_LAYER_FIRST,
        {"auto": B.KV_PATH_AUTO, "zerocopy": B.KV_PATH_ZEROCOPY, "sdma_staged": B.KV_PATH_SDMA_STAGED}[case["path"]],
        case["chunk_layers"],
        hbm_layout=B.KV_HBM_LAYER_FIRST if case["hbm_layout"] == "layer_first" else B.KV_HBM_BLOCK_FIRST)
    pinned = torch.empty(pool.numel(), dtype=torch.uint8, pin_memory=True)
    pinned.copy_(pool)
    del pool
    torch.cuda.synchronize()
    s = dict(kind=case["kind"], cfg=cfg, cache=cache, pool=pinned, out=(oi, os_), into=(ii, is_),
             outputs={"cache": _words(cache, case), "pool": _words(pinned, case)})
    if case["kind"] != "static":
        s["engine"] = B.Engine(cfg, cache.data_ptr(), pinned.data_ptr())
    if case["kind"] == "serve":
        # requests 0 and 1 take turns in HBM, request 2 is new in every iteration
        s["table"] = t = B.Table(s["engine"], 4)
        s["n_out"], s["grow"] = case["n_out"], case["n_out"] * case["tokens"]
        turn = case["n_in"] * case["tokens"]
        for call in (lambda: t.kv_table_append(0, turn)[0], lambda: t.kv_table_append(1, turn - 1)[0],
                     lambda: t.kv_table_rotate([1], []), lambda: t.kv_table_append(2, s["grow"])[0]):
            _ok(call())
        _ok(s["engine"].kv_wait())
    return s


def _ok(rc):
    if rc != 0:
        raise RuntimeError(B.kv_strerror(rc))


def run(s):
    kind = s["kind"]
    if kind == "static":
        stream = torch.cuda.current_stream()
        _ok(B.kv_rotate_static(s["cfg"], s["cache"].data_ptr(), s["pool"].data_ptr(), stream.cuda_stream,
                               *s["out"], *s["into"]))
        stream.synchronize()        # the pool may be read by the host from here on
        return s["outputs"]
    e = s["engine"]
    if kind == "reader":
        _ok(e.kv_reader_start(s["out"][0]))
        rc, checksum, _ = e.kv_reader_wait()
        _ok(rc)
        return {"checksum": np.array([checksum], dtype=np.uint64).view(np.int64)}
    if kind == "serve":
        t = s["table"]
        for leaves, returns in ((0, 1), (1, 0)):
            _ok(t.kv_table_rotate_eager([leaves], [returns], s["n_out"])[0])
            _ok(e.kv_wait())
            _ok(t.kv_table_finish(2))
            _ok(t.kv_table_append(2, s["grow"])[0])
        return s["outputs"]
    if kind == "rotate":
        _ok(e.kv_rotate(*s["out"], *s["into"]))
    elif kind == "swap_out":
        _ok(e.kv_swap_out(*s["out"]))
    else:
        _ok(e.kv_swap_in(s["into"][1], s["into"][0]))
    _ok(e.kv_wait())
    return s["outputs"]


def work(case):
    """Each byte moved is read once and written once; the reader only reads."""
    if case["kind"] == "reader":
        return {"bytes": case["n_out"] * _block(case), "flops": 0}
    times = 2 if case["kind"] == "serve" else 1
    return {"bytes": 2 * times * (case["n_out"] + case["n_in"]) * _block(case), "flops": 0}


def tolerance(case):
    return "exact"                  # bytes are moved, or summed as whole numbers


def exact(case, seed):
    if case["kind"] == "serve":     # where its blocks lie is the table's choice
        return None
    cache, pool, oi, os_, ii, is_ = _inputs(case, seed)
    nb, ns = _sizes(case)
    planes, cache, pool = 2 * case["layers"], _words(cache, case), _words(pool, case)
    # [plane, block or slot, word]
    c = cache.view(planes, nb, -1) if case["hbm_layout"] == "layer_first" else cache.view(nb, planes, -1).transpose(0, 1)
    p = pool.view(planes, ns, -1) if case["host_layout"] == "layer_first" else pool.view(ns, planes, -1).transpose(0, 1)
    at = [torch.from_numpy(a.astype(np.int64)).cuda() for a in (oi, os_, ii, is_)]
    if case["kind"] == "reader":
        total = sum(int((w.reshape(-1).view(torch.int32).to(torch.int64) & 0xFFFFFFFF).sum()) for w in c[:, at[0]])
        return {"checksum": np.array([total % (1 << 64)], dtype=np.uint64).view(np.int64)}
    out, into = c[:, at[0]].clone(), p[:, at[3]].clone()
    p[:, at[1]] = out
    c[:, at[2]] = into
    return {"cache": cache, "pool": pool.cpu()}

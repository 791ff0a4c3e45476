"""The transfers a program makes through this library, from one 4 KiB copy to the 64k-token KV fetch.

listed() names twelve of them, draw() gives more of the same ranges. prepare() builds what the
program holds before the call (pinned buffers, device tensors, block tables, the layer table),
run() makes the call or calls, and work() counts the bytes that have to move: every payload byte
is read once and written once. All outputs are copies of the inputs or modular sums over whole
words, so they are compared exactly.
"""
from __future__ import annotations

import ctypes
import math
import weakref

import numpy as np
import torch

import paper_2512_16056_amd as mma

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30
DIRS = {"h2d": mma.MMA_H2D, "d2h": mma.MMA_D2H}
LAYOUTS = {"piece": mma.MMA_KV_LAYOUT_PIECE, "xpacked": mma.MMA_KV_LAYOUT_XPACKED, "hnd": mma.MMA_KV_LAYOUT_HND}


def _kv(name, call, pool, layout, blocks, layers=32, tokens=16, heads=8, dim=128, elem=2):
    c = {"op": "kv", "call": call, "pool": pool, "layout": layout, "blocks": blocks, "layers": layers,
         "tokens": tokens, "heads": heads, "dim": dim, "elem": elem}
    return dict(c, name=name) if name else c


def listed():
    return [
        # Token ids, sampling parameters, one block table: the small copies of every decode step.
        {"name": "copy_h2d_4k", "op": "copy", "dir": "h2d", "bytes": 4 * KiB, "src_off": 0, "dst_off": 0},
        # Logits or hidden states brought to the host, of a size and at addresses nobody chose.
        {"name": "copy_d2h_ragged", "op": "copy", "dir": "d2h", "bytes": 1_000_003, "src_off": 16, "dst_off": 5},
        # The plain contiguous copy, 64 MiB.
        {"name": "copy_h2d_64m", "op": "copy", "dir": "h2d", "bytes": 64 * MiB, "src_off": 0, "dst_off": 0},
        # Model wake-up: four layers of the Llama-3-8B-shaped list, 36 tensors from 8 KiB to 112 MiB.
        {"name": "weights_wake_4_layers", "op": "weights", "dir": "h2d", "layers": 4, "hidden": 4096, "ffn": 14336,
         "kv_dim": 1024},
        # A prefix hit of one block (16 tokens): 64 pieces of 32 KiB.
        _kv("kv_fetch_1_block", "fetch", "host", "piece", 1),
        # The 64k-token prefix hit: 8 GiB in 262,144 pieces.
        _kv("kv_fetch_64k_tokens", "fetch", "host", "piece", 4096),
        # Eviction of 4k tokens from a cache in the layout of paged-attention decode kernels.
        _kv("kv_offload_xpacked", "offload", "host", "xpacked", 256),
        # A fetch inside a serving loop that must not allocate, head-major cache.
        _kv("kv_fetch_noalloc_hnd", "noalloc", "host", "hnd", 24),
        # The 64k-token fetch from a KV tier in this GPU's own memory.
        _kv("kv_hbm_fetch_64k_tokens", "fetch", "hbm", "piece", 4096),
        # Eviction of 8k tokens to the tier in HBM, head-major cache.
        _kv("kv_hbm_offload_hnd", "offload", "hbm", "hnd", 512),
        # A 16k-token hit in the tier in HBM, x-packed cache.
        _kv("kv_hbm_fetch_xpacked", "fetch", "hbm", "xpacked", 1024),
        # Mixed contention: two layers loaded and each checked by a dependent kernel on one stream,
        # while dirty KV blocks leave on another.
        {"name": "mixed_load_and_offload", "op": "mixed", "layers": 2, "hidden": 4096, "ffn": 14336, "kv_dim": 1024,
         "blocks": 256},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["copy", "copy", "weights", "kv", "kv", "kv", "kv", "kv", "mixed"])
    if op == "copy":
        n = _log(rng, 1 * KiB, 512 * MiB)
        if rng.random() < 0.5:
            n = max(1, n // (4 * KiB)) * 4 * KiB
            return {"op": "copy", "dir": rng.choice(["h2d", "d2h"]), "bytes": n, "src_off": 0, "dst_off": 0}
        return {"op": "copy", "dir": rng.choice(["h2d", "d2h"]), "bytes": n, "src_off": rng.randrange(64),
                "dst_off": rng.randrange(64)}
    if op in ("weights", "mixed"):
        hidden = rng.choice([768, 1024, 2048, 2560, 3072, 4096])
        ffn = rng.choice([4 * hidden, hidden * 7 // 2, hidden * 8 // 3 + 17])
        c = {"op": op, "layers": rng.randint(1, 4), "hidden": hidden, "ffn": ffn,
             "kv_dim": rng.choice([hidden, hidden // 4])}
        return dict(c, blocks=_log(rng, 4, 256)) if op == "mixed" else dict(c, dir=rng.choice(["h2d", "d2h"]))
    call = rng.choice(["fetch", "fetch", "offload", "noalloc"])
    pool = rng.choice(["host", "hbm"])
    layout = rng.choice(["piece", "xpacked", "hnd"])
    elem = rng.choice([1, 2, 2])
    tokens = rng.choice([16, 16, 32] if elem == 1 or layout != "piece" else [8, 16, 16, 32])
    shape = {"layers": rng.choice([2, 12, 24, 32, 36, 48]), "tokens": tokens, "heads": rng.choice([1, 2, 4, 5, 8]),
             "dim": rng.choice([64, 80, 96, 128, 128, 256]), "elem": elem}
    slot = 2 * shape["layers"] * tokens * shape["heads"] * shape["dim"] * elem
    top = (512 * MiB if pool == "host" else 4 * GiB) // slot
    return _kv(None, call, pool, layout, _log(rng, 1, max(2, min(top, 8192))), **shape)


# ------------------------------------------------------------------ inputs
_ready = False


def _init():
    global _ready
    if not _ready:
        torch.cuda.set_device(0)
        mma.mma_init(0)
        _ready = True


def _host(nbytes):
    """Pinned host memory of the library as a uint8 array; freed with its last view."""
    n = (nbytes + 4095) // 4096 * 4096
    raw = (ctypes.c_uint8 * n).from_address(mma.mma_host_alloc(n))
    weakref.finalize(raw, mma.mma_host_free, ctypes.addressof(raw))
    return np.frombuffer(raw, np.uint8)


def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _random(nbytes, g):
    """Random bytes on the GPU (KV values and payloads as a copy sees them)."""
    return torch.empty((nbytes + 7) // 8, dtype=torch.int64, device="cuda").random_(generator=g).view(torch.uint8)


def _perm(n, take, g):
    return torch.randperm(n, generator=g, device="cuda")[:take].to(torch.int32).cpu().numpy()


def _fill_host(array, gpu_bytes):
    torch.from_numpy(array[: gpu_bytes.numel()]).copy_(gpu_bytes)


def _padded(nbytes):
    return (nbytes + 64 + 4095) // 4096 * 4096


def _weight_sizes(c):
    """Bytes of the nine bf16 tensors of each layer, in load order."""
    h, f, k = c["hidden"], c["ffn"], c["kv_dim"]
    return [2 * n for _ in range(c["layers"]) for n in (h, h * h, k * h, k * h, h * h, h, f * h, f * h, h * f)]


def _offsets(sizes):
    offs, cur = [], 0
    for s in sizes:
        offs.append(cur)
        cur += (s + 255) // 256 * 256
    return offs, cur


def _weights(c, direction, g):
    """(copies, host arena, device arena): bf16 N(0, 0.02) weights on the side they are loaded from."""
    sizes = _weight_sizes(c)
    offs, total = _offsets(sizes)
    vals = torch.empty(total // 2, dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=g)
    vals = vals.view(torch.uint8)
    host = _host(total)
    if direction == "h2d":
        _fill_host(host, vals)
        dev = torch.zeros(total, dtype=torch.uint8, device="cuda")
    else:
        host[:] = 0
        dev = vals
    hp, dp = host.ctypes.data, dev.data_ptr()
    if direction == "h2d":
        copies = [(dp + o, hp + o, s) for o, s in zip(offs, sizes)]
    else:
        copies = [(hp + o, dp + o, s) for o, s in zip(offs, sizes)]
    return copies, host, dev


def _kv_shape(c):
    piece = c["tokens"] * c["heads"] * c["dim"] * c["elem"]
    n = c["blocks"]
    gpu_blocks = n + n // 16 + 1
    slots = 2 * n if c["call"] == "offload" else n
    return piece, gpu_blocks, slots


def _kv_state(c, g):
    piece, nb, slots = _kv_shape(c)
    lay = mma.kv_layout(c["layers"], c["tokens"], c["heads"], c["dim"], c["elem"], nb, slots, LAYOUTS[c["layout"]])
    pool_bytes, cache_bytes = slots * 2 * c["layers"] * piece, c["layers"] * 2 * nb * piece
    offload = c["call"] == "offload"
    cache = _random(cache_bytes, g) if offload else torch.zeros(cache_bytes, dtype=torch.uint8, device="cuda")
    if c["pool"] == "hbm":
        pool = torch.zeros(pool_bytes, dtype=torch.uint8, device="cuda") if offload else _random(pool_bytes, g)
    else:
        pool = _host(pool_bytes)
        if offload:
            pool[:] = 0
        else:
            _fill_host(pool, _random(pool_bytes, g))
    table = mma.layer_table(list(cache.view(c["layers"], -1)))
    out = cache if not offload else pool
    return {"layout": lay, "pool": pool, "cache": cache, "table": table,
            "slots": _perm(slots, c["blocks"], g), "gpu_blocks": _perm(nb, c["blocks"], g),
            "out": out.view(torch.int64 if isinstance(out, torch.Tensor) else np.int64)}


def prepare(case, seed):
    _init()
    g = _rng(seed)
    if case["op"] == "copy":
        src_bytes, dst_bytes = _padded(case["bytes"]), _padded(case["bytes"])
        data = _random(src_bytes, g)
        host = _host(src_bytes)
        if case["dir"] == "h2d":
            _fill_host(host, data)
            dev = torch.zeros(dst_bytes, dtype=torch.uint8, device="cuda")
            dst, src, out = dev.data_ptr(), host.ctypes.data, dev.view(torch.int64)
        else:
            host[:] = 0
            dev = data
            dst, src, out = host.ctypes.data, dev.data_ptr(), host.view(np.int64)
        return {"run": _run_copy, "dst": dst + case["dst_off"], "src": src + case["src_off"], "bytes": case["bytes"],
                "dir": DIRS[case["dir"]], "host": host, "dev": dev, "out": out}
    if case["op"] == "weights":
        copies, host, dev = _weights(case, case["dir"], g)
        out = dev.view(torch.int64) if case["dir"] == "h2d" else host.view(np.int64)
        return {"run": _run_weights, "copies": copies, "dir": DIRS[case["dir"]], "host": host, "dev": dev, "out": out}
    if case["op"] == "kv":
        s = _kv_state(case, g)
        s["run"] = {"fetch": _run_fetch, "noalloc": _run_noalloc, "offload": _run_offload}[case["call"]]
        return s
    copies, host, dev = _weights(case, "h2d", g)
    kv = _kv_state(_mixed_kv(case), g)
    groups = [copies[i: i + 9] for i in range(0, len(copies), 9)]
    spans = [(grp[0][0], grp[-1][0] + grp[-1][2] - grp[0][0]) for grp in groups]
    return {"run": _run_mixed, "groups": groups, "spans": spans, "host": host, "dev": dev, "kv": kv,
            "digest": torch.zeros(len(groups), dtype=torch.int64, device="cuda"),
            "load": torch.cuda.Stream(), "evict": torch.cuda.Stream(), "out": dev.view(torch.int64)}


def _mixed_kv(c):
    return _kv(None, "offload", "host", "piece", c["blocks"])


# ------------------------------------------------------------------ one pass
def _run_copy(s):
    mma.mma_memcpy_async(s["dst"], s["src"], s["bytes"], s["dir"])
    return s["out"]


def _run_weights(s):
    mma.mma_weights_load(s["copies"], s["dir"])
    return s["out"]


def _run_fetch(s):
    mma.mma_kv_fetch(s["layout"], s["pool"], s["table"], s["slots"], s["gpu_blocks"])
    return s["out"]


def _run_noalloc(s):
    mma.mma_kv_fetch_noalloc(s["layout"], s["pool"], s["table"], s["slots"], s["gpu_blocks"])
    return s["out"]


def _run_offload(s):
    mma.mma_kv_offload(s["layout"], s["pool"], s["table"], s["gpu_blocks"], s["slots"])
    return s["out"]


def _run_mixed(s):
    kv = s["kv"]
    here = torch.cuda.current_stream()
    s["load"].wait_stream(here)
    s["evict"].wait_stream(here)
    mma.mma_kv_offload(kv["layout"], kv["pool"], kv["table"], kv["gpu_blocks"], kv["slots"], s["evict"])
    with torch.cuda.stream(s["load"]):
        s["digest"].zero_()
        for i, (grp, (ptr, n)) in enumerate(zip(s["groups"], s["spans"])):
            mma.mma_weights_load(grp, mma.MMA_H2D)
            mma.mma_digest_u32(ptr, n // 4 * 4, s["digest"].data_ptr() + 8 * i)
    here.wait_stream(s["load"])
    here.wait_stream(s["evict"])
    return {"weights": s["out"], "digest": s["digest"], "pool": kv["out"]}


def run(state):
    return state["run"](state)


# ------------------------------------------------------------------ work and results
def work(case):
    if case["op"] == "copy":
        return {"bytes": 2 * case["bytes"], "flops": 0}
    if case["op"] == "kv":
        return {"bytes": 2 * case["blocks"] * 2 * case["layers"] * _kv_shape(case)[0], "flops": 0}
    total = 2 * sum(_weight_sizes(case))
    if case["op"] == "mixed":  # the check kernel reads each loaded group once
        total += total // 2 + work(_mixed_kv(case))["bytes"]
    return {"bytes": total, "flops": 0}


def tolerance(case):
    return "exact"


def _to_block(pieces, c):
    """[..., tokens, heads, dim, elem] pieces (two: K and V, on axis 1) as GPU blocks."""
    if c["layout"] == "piece":
        return pieces.flatten(2)
    if c["layout"] == "hnd":
        return pieces.permute(0, 1, 3, 2, 4, 5).flatten(2)
    x = 16 // c["elem"]
    n, t, h, d, e = pieces.shape[0], c["tokens"], c["heads"], c["dim"], c["elem"]
    k = pieces[:, 0].reshape(n, t, h, d // x, x, e).permute(0, 2, 3, 1, 4, 5).flatten(1)
    v = pieces[:, 1].permute(0, 2, 3, 1, 4).flatten(1)
    return torch.stack([k, v], 1)


def _from_block(blocks, c):
    """The inverse of _to_block: [n, 2, piece bytes] -> [n, 2, piece bytes] token-major."""
    n, t, h, d, e = blocks.shape[0], c["tokens"], c["heads"], c["dim"], c["elem"]
    if c["layout"] == "piece":
        return blocks
    if c["layout"] == "hnd":
        return blocks.view(n, 2, h, t, d, e).permute(0, 1, 3, 2, 4, 5).flatten(2)
    x = 16 // e
    k = blocks[:, 0].view(n, h, d // x, t, x, e).permute(0, 3, 1, 2, 4, 5).flatten(1)
    v = blocks[:, 1].view(n, h, d, t, e).permute(0, 3, 1, 2, 4).flatten(1)
    return torch.stack([k, v], 1)


def _gpu(x):
    return x if isinstance(x, torch.Tensor) else torch.from_numpy(x).cuda()


def _exact_kv(s, c):
    piece, nb, slots = _kv_shape(c)
    pool = _gpu(s["pool"])[: slots * 2 * c["layers"] * piece].view(slots, c["layers"], 2, piece)
    cache = s["cache"].view(c["layers"], 2, nb, piece)
    hs, gb = (torch.from_numpy(a).long().cuda() for a in (s["slots"], s["gpu_blocks"]))
    shape = (len(hs), 2, c["tokens"], c["heads"], c["dim"], c["elem"])
    if c["call"] != "offload":
        out = torch.zeros_like(cache)
        for l in range(c["layers"]):
            out[l][:, gb] = _to_block(pool[hs, l].view(shape), c).transpose(0, 1)
        return out.flatten().view(torch.int64)
    out = torch.zeros_like(pool)
    for l in range(c["layers"]):
        out[hs, l] = _from_block(cache[l][:, gb].transpose(0, 1).contiguous(), c)
    flat = torch.zeros(len(s["out"]) * 8, dtype=torch.uint8, device="cuda")
    flat[: out.numel()] = out.flatten()
    flat = flat.view(torch.int64)
    return flat if c["pool"] == "hbm" else flat.cpu().numpy()


def exact(case, seed):
    """What run() returns, by plain indexing and integer arithmetic."""
    s = prepare(case, seed)
    if case["op"] == "copy":
        host, dev = torch.from_numpy(s["host"]), s["dev"].cpu()
        src, dst = (host, dev) if case["dir"] == "h2d" else (dev, host)
        out = torch.zeros_like(dst)
        out[case["dst_off"]: case["dst_off"] + case["bytes"]] = \
            src[case["src_off"]: case["src_off"] + case["bytes"]]
        return out.view(torch.int64) if case["dir"] == "h2d" else out.view(torch.int64).numpy()
    if case["op"] == "kv":
        return _exact_kv(s, case)
    sizes = _weight_sizes(case)
    offs, total = _offsets(sizes)
    h2d = case["op"] == "mixed" or case["dir"] == "h2d"
    src = torch.from_numpy(s["host"])[:total] if h2d else s["dev"].cpu()
    out = torch.zeros(total if h2d else len(s["host"]), dtype=torch.uint8)
    for o, n in zip(offs, sizes):
        out[o: o + n] = src[o: o + n]
    if case["op"] == "weights":
        return out.view(torch.int64) if h2d else out.view(torch.int64).numpy()
    digests = []
    for g in range(case["layers"]):
        a, b = offs[9 * g], offs[9 * g + 8] + sizes[9 * g + 8]
        w = out[a: a + (b - a) // 4 * 4].view(torch.int32).cuda().long() & 0xFFFFFFFF
        i = torch.arange(w.numel(), device="cuda")
        digests.append(((w + 1) * (2 * i + 1)).sum())  # int64 arithmetic wraps modulo 2^64
    return {"weights": out.view(torch.int64), "digest": torch.stack(digests),
            "pool": _exact_kv(s["kv"], _mixed_kv(case))}

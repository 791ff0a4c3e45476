"""Benchmark of the multipath host->GPU path on one MI355X.

One step = one paged-KV fetch of a 64k-token prompt prefix (Llama-3-8B GQA shape:
32 layers x K,V x 8 kv heads x 128 dims, bf16, 16-token blocks -> 4096 blocks,
8 GiB) from a pinned host pool into the GPU's paged cache through
mma_kv_fetch. The step exercises every part of the path: planner, CU-path
gather, SDMA staging + HBM scatter, completion counters and the stream wait.
Inputs are resident (host pool filled, GPU cache allocated) before timing.

Printed: one JSON line (stdout) with the throughput, the KV fetch latency, the
roofline of the dummy-task kernel (PCIe-bound), the oracle's CPU throughput on
the same workload, native hipMemcpyAsync comparators, and the 64 MiB single-copy
workload.

Usage: python bench.py [--gpus 1] [--steps 10] [--warmup 2]
       python bench.py --sweep sizes|idle|blocking|chunks|contention|duplex|paths|footprint|control|hbmpool|misaligned|mixed
                                                                (JSON per point)
       python bench.py --calib                                  (counter-scaling kernels)
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time
from concurrent.futures import ThreadPoolExecutor

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "host→GPU GB/s per copy (% of PCIe5 x16 peak); 64k-token KV fetch latency"
PCIE5_X16_GBS = 32e9 * 16 * 128 / 130 / 8 / 1e9   # 63.0 GB/s per direction after 128b/130b coding


def log(*a):
    print(*a, file=sys.stderr, flush=True)


_ENGINE_NAP_US = None  # --engine-nap-us


def _default_config():
    """The library's default configuration, with --engine-nap-us applied."""
    import paper_2512_16056_amd as mma
    c = mma.mma_config_default()
    if _ENGINE_NAP_US is not None:
        c.engine_nap_us = _ENGINE_NAP_US
    return c


def parse():
    p = argparse.ArgumentParser()
    p.add_argument("--gpus", type=int, default=int(os.environ.get("WORLD_SIZE", "1")))
    p.add_argument("--steps", type=int, default=10)
    p.add_argument("--warmup", type=int, default=2)
    p.add_argument("--kv-layout", choices=["piece", "xpacked", "hnd"], default="piece",
                   help="GPU block layout of the timed KV fetch: pieces as in host memory (default), the "
                        "x-packed layout of paged-attention decode kernels (transformed through LDS), or "
                        "head-major blocks [heads][tokens][head_dim] (a row permutation)")
    p.add_argument("--no-cpu-baseline", action="store_true")
    p.add_argument("--no-extras", action="store_true", help="skip native comparators and the 64 MiB copy")
    p.add_argument("--cpu-seconds", type=float, default=10.0, help="minimum oracle timing window")
    p.add_argument("--control", choices=["host", "device"], default=None,
                   help="who drives transfers after submission (default: the library's, MMA_CONTROL)")
    p.add_argument("--sweep", choices=["sizes", "idle", "chunks", "contention", "duplex", "paths", "footprint",
                                       "control", "hbmpool", "misaligned", "mixed", "blocking"],
                   help="instead of the benchmark, print one JSON line per point of a parameter sweep")
    p.add_argument("--oracle-cores", default=None,
                   help=argparse.SUPPRESS)  # the all-cores oracle baseline's worker process (CPU only)
    p.add_argument("--sizes", default=None,
                   help="comma-separated transfer sizes in bytes for --sweep idle (default: 32 KiB to 8 GiB) "
                        "or --sweep blocking (default: 64 KiB to 64 MiB)")
    p.add_argument("--calib", action="store_true",
                   help="only run plain kernels of known traffic (1 GiB fill, read, copy) for counter scaling")
    p.add_argument("--engine-nap-us", type=int, default=None,
                   help="engine_nap_us of every configuration the run uses (default: the library's; "
                        "4294967295 = MMA_ENGINE_NAP_OFF, the engine threads poll without sleeping)")
    return p.parse_args()


def calibration_kernels():
    """Plain kernels of known HBM traffic, run under rocprofv3 --pmc to scale FETCH_SIZE/WRITE_SIZE:
    a torch fill (writes N), mma_digest_u32 (reads N) and a device-to-device copy (reads N, writes N)."""
    import torch

    import paper_2512_16056_amd as mma
    n = 1 << 30
    mma.mma_init(0)
    a = torch.empty(n, dtype=torch.uint8, device="cuda")
    b = torch.empty(n, dtype=torch.uint8, device="cuda")
    out = torch.zeros(1, dtype=torch.int64, device="cuda")
    for _ in range(3):
        a.fill_(7)
        mma.mma_digest_u32(a, n, out)
        b.copy_(a)
    torch.cuda.synchronize()
    mma.mma_finalize()
    print(json.dumps({"calibration": {"bytes": n, "kernels": ["fill: write N", "mma_digest_kernel: read N",
                                                              "copyBuffer: read N + write N"]}}), flush=True)


# Every source file that the device code is compiled from, in a fixed order.
KERNEL_SOURCES = ("mma_kernels.hip", "mma_proto.h", "mma_xpacked.h", "mma_pool.h")


def kernel_sources_sha256(root: str) -> str:
    """SHA-256 over the device sources (each file's bytes, in KERNEL_SOURCES order)."""
    import hashlib
    h = hashlib.sha256()
    for name in KERNEL_SOURCES:
        with open(os.path.join(root, "paper_2512_16056_amd", "csrc", name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def recorded_traffic(root: str, kernel: str = "mma_transfer_kernel"):
    """HBM/EA bytes per launch of the transfer kernel from the committed rocprofv3 --pmc summary,
    valid only while the device sources are the ones that were profiled."""
    path = os.path.join(root, "profiles", f"{kernel}__kv_fetch_64k.traffic.json")
    try:
        rec = json.load(open(path))
        sha = kernel_sources_sha256(root)
    except (OSError, ValueError):
        return None
    if rec.get("kernel_sources_sha256") != sha:
        return None
    return rec.get("traffic_bytes_per_launch")


def _timed(stream, fn, reps, warm):
    """Median (and p10/p90) of HIP-event-bracketed runs of fn on `stream`."""
    import torch
    for _ in range(warm):
        fn()
    stream.synchronize()
    ts = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(stream)
        fn()
        b.record(stream)
        b.synchronize()
        ts.append(a.elapsed_time(b))
    return _pcts(ts)


def _ok(rc):
    if rc != 0:
        raise RuntimeError(f"library call failed with status {rc}")


def _pcts(ts):
    ts = sorted(ts)

    def q(p):
        return ts[min(len(ts) - 1, int(round(p * (len(ts) - 1))))]
    return {"p10": q(0.1), "p50": q(0.5), "p90": q(0.9), "mean": sum(ts) / len(ts), "n": len(ts)}


def native_lib():
    import ctypes
    nat = ctypes.CDLL(os.path.join(ROOT, "paper_2512_16056_amd", "libmma_native.so"))
    vp, u64, u32, i32 = ctypes.c_void_p, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int
    kv_args = [vp, vp, vp, vp, u64, u32, u64, u64, vp]
    for name, args in (("native_kv_fetch", kv_args), ("native_kv_fetch_batch", kv_args),
                       ("native_kv_offload", kv_args), ("native_list", [vp, vp, vp, u64, i32, vp]),
                       ("native_zero_copy", [vp, vp, u64, i32, u32, vp]),
                       ("native_hbm_copy", [vp, vp, u64, u32, vp]),
                       ("native_sdma_all", [vp, vp, u64, i32, u32, i32, ctypes.POINTER(u64)])):
        fn = getattr(nat, name)
        fn.restype = ctypes.c_int
        fn.argtypes = args
    return nat


def link_peaks(mma, nat, stream, sdma_mask):
    """Measured link peak M(dir): the best of three raw 1 GiB probes that bypass the multipath
    planner -- one hipMemcpyAsync (median of 20), every host-facing SDMA engine at once over equal
    parts (median of 5), and a bare zero-copy streaming kernel at the best grid of a sweep
    (median of 3 per grid)."""
    import ctypes

    import torch
    n = 1 << 30
    hbuf = mma.PinnedBuffer(n)
    hbuf.array[::4096] = 1
    dbuf = torch.empty(n, dtype=torch.uint8, device="cuda")
    res = {}
    for d, name in ((0, "h2d"), (1, "d2h")):
        dst, src = (dbuf.data_ptr(), hbuf.ptr) if d == 0 else (hbuf.ptr, dbuf.data_ptr())
        D, S, Z = (ctypes.c_void_p * 1)(dst), (ctypes.c_void_p * 1)(src), (ctypes.c_uint64 * 1)(n)
        memcpy = _timed(stream, lambda: nat.native_list(D, S, Z, 1, d, ctypes.c_void_p(stream.cuda_stream)),
                        reps=20, warm=2)["p50"]
        torch.cuda.synchronize()
        ns = ctypes.c_uint64(0)
        sd = []
        for _ in range(6):
            rc = nat.native_sdma_all(dst, src, n, d, sdma_mask, 0, ctypes.byref(ns))
            if rc != 0:
                sd = []
                break
            sd.append(ns.value / 1e6)
        sdma = _pcts(sd[1:])["p50"] if sd else None
        zc = {}
        for grid in (16, 32, 64, 128, 256, 512, 1024):
            zc[grid] = _timed(stream, lambda: nat.native_zero_copy(dst, src, n, d, grid,
                                                                   ctypes.c_void_p(stream.cuda_stream)),
                              reps=3, warm=1)["p50"]
        best_grid = min(zc, key=zc.get)
        rates = {"hipMemcpyAsync": n / memcpy / 1e6, "sdma_all": n / sdma / 1e6 if sdma else None,
                 "zero_copy_kernel": n / zc[best_grid] / 1e6}
        res[name] = {"peak_GBs": round(max(v for v in rates.values() if v), 2),
                     **{k: (round(v, 2) if v else None) for k, v in rates.items()},
                     "zero_copy_best_grid": best_grid,
                     "sdma_mask": hex(sdma_mask)}
    # Both directions at once: one hipMemcpyAsync of 1 GiB each way on two streams (median of 3);
    # the aggregate is the reference for transfers that overlap in both directions.
    hbuf2 = mma.PinnedBuffer(n)
    hbuf2.array[::4096] = 1
    dbuf2 = torch.empty(n, dtype=torch.uint8, device="cuda")
    s2 = torch.cuda.Stream()
    D1, S1, Z = (ctypes.c_void_p * 1)(dbuf.data_ptr()), (ctypes.c_void_p * 1)(hbuf.ptr), (ctypes.c_uint64 * 1)(n)
    D2, S2 = (ctypes.c_void_p * 1)(hbuf2.ptr), (ctypes.c_void_p * 1)(dbuf2.data_ptr())
    agg = []
    for _ in range(4):
        torch.cuda.synchronize()
        e = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        e[0].record(stream)
        e[2].record(s2)
        nat.native_list(D1, S1, Z, 1, 0, ctypes.c_void_p(stream.cuda_stream))
        nat.native_list(D2, S2, Z, 1, 1, ctypes.c_void_p(s2.cuda_stream))
        e[1].record(stream)
        e[3].record(s2)
        torch.cuda.synchronize()
        agg.append(n / e[0].elapsed_time(e[1]) / 1e6 + n / e[2].elapsed_time(e[3]) / 1e6)
    res["duplex_GBs"] = round(sorted(agg[1:])[1], 2)
    del dbuf, dbuf2
    hbuf.free()
    hbuf2.free()
    return res


def gpu_local_cpus(torch):
    """(NUMA node, its CPUs) of GPU 0, from sysfs; (None, []) when unknown."""
    p = torch.cuda.get_device_properties(0)
    dev = f"/sys/bus/pci/devices/{p.pci_domain_id:04x}:{p.pci_bus_id:02x}:{p.pci_device_id:02x}.0"
    try:
        node = int(open(os.path.join(dev, "numa_node")).read().strip())
        cpus = []
        for part in open(os.path.join(dev, "local_cpulist")).read().strip().split(","):
            a, _, b = part.partition("-")
            cpus.extend(range(int(a), int(b or a) + 1))
        return node, cpus
    except (OSError, ValueError):
        return None, []


# One GPU's job on these hosts gets a 16-CPU share of the machine, whatever the node holds.
HOST_CPU_SHARE = 16


def oracle_all_cores(torch, seconds):
    """The oracle KV fetch spread over one process per core: the CPUs of the GPU's NUMA node that
    this process may use (at most the job's CPU share), each process pinned to one of them and
    working on its own disjoint slices of the 4096-entry block table (64 blocks x one layer per
    call). Aggregate payload GB/s over the slowest worker's time."""
    import subprocess
    node, local = gpu_local_cpus(torch)
    allowed = sorted(os.sched_getaffinity(0))
    use = [c for c in local if c in set(allowed)] or allowed
    use = use[:HOST_CPU_SHARE]
    r = subprocess.run([sys.executable, os.path.abspath(__file__), "--oracle-cores", ",".join(map(str, use)),
                        "--cpu-seconds", str(seconds)], capture_output=True, text=True, timeout=600)
    lines = [x for x in r.stdout.splitlines() if x.startswith("{")]
    if r.returncode != 0 or not lines:
        return {"value": None, "error": f"exit {r.returncode}: {r.stderr[-300:]}"}
    res = json.loads(lines[-1])
    res.update({"numa_node": node, "node_cpus": len(local), "cpus_allowed": len(allowed),
                "cpu_share_cap": HOST_CPU_SHARE})
    return res


def oracle_cores_worker(cores, seconds):
    """Child of oracle_all_cores (no GPU in this process): a pageable copy of the pool's shape,
    then one forked worker per core, released together, each running oracle.kv.kv_fetch_layer
    over its own (layer, 64-block slice) tasks until the deadline; one JSON line."""
    import numpy as np

    import workloads as W
    from oracle import kv as okv
    s = W.KV64K
    hs, _ = W.kv_fetch_tables(s, cfg=3)
    pool = np.empty((s.host_num_slots, s.slot_bytes), np.uint8)
    with ThreadPoolExecutor(len(cores)) as ex:  # touch every page before the workers fork
        list(ex.map(lambda i: pool[i:i + 64].fill(0x3C), range(0, s.host_num_slots, 64)))
    span = 64
    tasks = [(l, a) for l in range(s.layers) for a in range(0, s.n_blocks, span)]
    poison = np.full((2, span, s.piece_bytes), W.GPU_POISON, np.uint8)
    local_blocks = np.arange(span, dtype=np.int32)
    go_r, go_w = os.pipe()
    res_r, res_w = os.pipe()
    kids = []
    for k, core in enumerate(cores):
        pid = os.fork()
        if pid == 0:
            os.close(go_w)
            os.close(res_r)
            os.sched_setaffinity(0, {core})
            mine = tasks[k::len(cores)]
            okv.kv_fetch_layer(pool, poison, mine[0][0], s.layers, hs[mine[0][1]:mine[0][1] + span], local_blocks)
            os.read(go_r, 1)  # released together
            t0 = time.perf_counter()
            done = 0
            while True:
                for l, a in mine:
                    okv.kv_fetch_layer(pool, poison, l, s.layers, hs[a:a + span], local_blocks)
                    done += span * 2 * s.piece_bytes
                if time.perf_counter() - t0 >= seconds:
                    break
            os.write(res_w, f"{done} {time.perf_counter() - t0}\n".encode())
            os._exit(0)
        kids.append(pid)
    os.close(go_r)
    os.close(res_w)
    os.write(go_w, b"x" * len(cores))
    out = b""
    while True:
        chunk = os.read(res_r, 4096)
        if not chunk:
            break
        out += chunk
    for pid in kids:
        os.waitpid(pid, 0)
    rows = [x.split() for x in out.decode().splitlines() if x.strip()]
    moved = sum(int(a) for a, _ in rows)
    wall = max(float(b) for _, b in rows)
    print(json.dumps({"value": round(moved / wall / 1e9, 3), "unit": "GB/s", "cores": len(rows), "kind": "oracle",
                      "cpus": cores, "sample": f"{moved / s.slot_bytes / s.n_blocks:.1f} x the 64k-token fetch "
                      f"(oracle.kv.kv_fetch_layer on (layer, 64-block) slices of the table), {len(rows)} processes "
                      f"pinned one per CPU, {wall:.1f} s"}), flush=True)


def run_native_batch(s, hs, gb):
    """One hipMemcpyBatchAsync of the 262,144 pieces of the 64k-token fetch, from the standalone
    comparator program (it links the system ROCm runtime, which exports the call), run as its
    own process with the same block tables. Its JSON line, or the reason it has none."""
    import subprocess
    import tempfile

    import numpy as np
    exe = os.path.join(ROOT, "paper_2512_16056_amd", "native_batch")
    if not os.path.exists(exe):
        return {"available": False, "error": "native_batch not built"}
    with tempfile.NamedTemporaryFile(suffix=".i32", delete=False) as f:
        f.write(np.concatenate([hs, gb]).astype(np.int32).tobytes())
        path = f.name
    try:
        r = subprocess.run([exe, path, str(s.n_blocks), str(s.layers), str(s.piece_bytes), str(s.gpu_num_blocks),
                            str(s.host_num_slots), "3"], capture_output=True, text=True, timeout=300)
    except subprocess.TimeoutExpired:
        return {"available": False, "error": "timed out after 300 s"}
    finally:
        os.unlink(path)
    if r.returncode < 0 or r.returncode >= 128:
        # the comparator died (a signal, e.g. a fault): touch the GPU no further in this process
        raise SystemExit(f"native_batch ended with status {r.returncode}: {r.stderr[-500:]}")
    lines = [x for x in r.stdout.splitlines() if x.startswith("{")]
    if r.returncode != 0 or not lines:
        return {"available": False, "error": f"exit {r.returncode}: {(r.stderr or r.stdout)[-300:]}"}
    return json.loads(lines[-1])


def run_extras(mma, W, np, torch, s, pool, layers, lay, hs, gb, stream, ms_per_step, total, out,
               native_batch=None):
    import ctypes
    extras = {}
    nat = native_lib()
    cfg = mma.mma_get_config().as_dict()

    peaks = link_peaks(mma, nat, stream, cfg["path_mask_h2d"] & 0xFFFF)
    extras["measured_link"] = peaks
    m_h2d, m_d2h = peaks["h2d"]["peak_GBs"], peaks["d2h"]["peak_GBs"]
    out["roofline"]["measured_peak"] = m_h2d
    out["roofline"]["frac_of_measured"] = round(out["roofline"]["achieved"] / m_h2d, 4)
    log("measured link:", peaks)

    # native KV fetch comparators: (n1) 262,144 per-piece hipMemcpyAsync calls, host-timed from the
    # first call to the stream's completion; (n2) one hipMemcpyBatchAsync with the same 262,144
    # entries, event-timed in its own process (run_native_batch). "Native" is the best of the two.
    lp = (ctypes.c_void_p * s.layers)(*[t.data_ptr() for t in layers])
    hs_c, gb_c = hs.ctypes.data_as(ctypes.c_void_p), gb.ctypes.data_as(ctypes.c_void_p)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    rc = nat.native_kv_fetch(pool.ptr, lp, hs_c, gb_c, s.n_blocks, s.layers, s.piece_bytes, s.gpu_num_blocks,
                             ctypes.c_void_p(stream.cuda_stream))
    stream.synchronize()
    extras["native_kv_fetch_ms"] = round((time.perf_counter() - t0) * 1e3, 2) if rc == 0 else None
    nb = native_batch or {"available": False, "error": "not run"}
    extras["native_kv_fetch_batch"] = nb
    extras["native_kv_fetch_batch_ms"] = nb.get("ms_median") if nb.get("ok") else None
    natives = [v for v in (extras["native_kv_fetch_ms"], extras["native_kv_fetch_batch_ms"]) if v]
    if natives:
        extras["native_kv_fetch_best_ms"] = min(natives)
        extras["kv_fetch_speedup_vs_native"] = round(min(natives) / ms_per_step, 3)

    # the 64 MiB single-copy workload: MMA vs one hipMemcpyAsync, 50 runs each after 5 warm-ups
    n = W.COPY64_BYTES
    src = mma.PinnedBuffer(n)
    src.array[:] = W.uniform_bytes(1, W.TAG_DATA, 0, n)
    dst = torch.full((n,), W.WEIGHT_POISON, dtype=torch.uint8, device="cuda")
    # Both sides are called straight through ctypes with prepared arguments, so neither pays
    # Python-level argument conversion inside the timed region.
    margs = (ctypes.c_void_p(dst.data_ptr()), ctypes.c_void_p(src.ptr), ctypes.c_uint64(n), mma.MMA_H2D,
             ctypes.c_void_p(stream.cuda_stream))
    m64 = _timed(stream, lambda: _ok(mma.lib.mma_memcpy_async(*margs)), reps=50, warm=5)
    ok64 = bool(np.array_equal(dst.cpu().numpy(), src.array))
    D, S, Z = (ctypes.c_void_p * 1)(dst.data_ptr()), (ctypes.c_void_p * 1)(src.ptr), (ctypes.c_uint64 * 1)(n)
    sp = ctypes.c_void_p(stream.cuda_stream)
    n64 = _timed(stream, lambda: nat.native_list(D, S, Z, 1, 0, sp), reps=50, warm=5)
    extras["copy64"] = {"mma_ms": round(m64["p50"], 4), "mma_ms_p10_p90": [round(m64["p10"], 4), round(m64["p90"], 4)],
                        "mma_GBs": round(n / m64["p50"] / 1e6, 2),
                        "native_ms": round(n64["p50"], 4),
                        "native_ms_p10_p90": [round(n64["p10"], 4), round(n64["p90"], 4)],
                        "native_GBs": round(n / n64["p50"] / 1e6, 2),
                        "ratio_vs_native": round(n64["p50"] / m64["p50"], 3), "parity": ok64,
                        "frac_of_pcie5": round(n / m64["p50"] / 1e6 / PCIE5_X16_GBS, 4),
                        "frac_of_measured": round(n / m64["p50"] / 1e6 / m_h2d, 4)}
    src.free()
    del dst

    # KV offload (GPU -> host): the 50%-dirty subset of the cache just fetched, 2048 blocks (4 GiB),
    # into a permutation of host slots; against 131,072 per-piece hipMemcpyAsync D2H.
    plan = W.kv_offload_plan(s, cfg=4)
    src_blocks = gb[plan.dirty].astype(np.int32)
    off_bytes = len(plan.dirty) * s.slot_bytes
    off = _timed(stream, lambda: mma.mma_kv_offload(lay, pool, layers, src_blocks, plan.dest, stream), reps=5, warm=1)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    rc = nat.native_kv_offload(pool.ptr, lp, src_blocks.ctypes.data_as(ctypes.c_void_p),
                               plan.dest.ctypes.data_as(ctypes.c_void_p), len(plan.dirty), s.layers, s.piece_bytes,
                               s.gpu_num_blocks, ctypes.c_void_p(stream.cuda_stream))
    stream.synchronize()
    nat_off = (time.perf_counter() - t0) * 1e3 if rc == 0 else None
    extras["kv_offload_2048_blocks"] = {
        "mma_ms": round(off["p50"], 3), "mma_ms_p10_p90": [round(off["p10"], 3), round(off["p90"], 3)],
        "mma_GBs": round(off_bytes / off["p50"] / 1e6, 2),
        "frac_of_measured_d2h": round(off_bytes / off["p50"] / 1e6 / m_d2h, 4),
        "native_per_piece_ms": round(nat_off, 2) if nat_off else None,
        "speedup_vs_native": round(nat_off / off["p50"], 2) if nat_off else None}

    # The same 64k-token fetch, and the 2048-block offload, with the GPU cache in the x-packed block
    # layout of paged-attention decode kernels (key [H][D/x][B][x], value [H][D][B]): the CU path
    # transforms every piece through LDS. Sampled parity against the layout's definition.
    # The same fetch and offload into the transformed GPU block layouts.
    pv = pool.array.reshape(s.host_num_slots, s.slot_bytes)
    for key, code in (("kv_xpacked_layout", mma.MMA_KV_LAYOUT_XPACKED), ("kv_hnd_layout", mma.MMA_KV_LAYOUT_HND)):
        xlay = mma.kv_layout(s.layers, s.block_tokens, s.kv_heads, s.head_dim, s.elem_bytes, s.gpu_num_blocks,
                             s.host_num_slots, code)
        xf = _timed(stream, lambda: mma.mma_kv_fetch(xlay, pool, layers, hs, gb, stream), reps=5, warm=1)
        ok_x = sampled_fetch_parity(s, pv, layers, hs, gb, code, samples=32, seed=1)
        xo = _timed(stream, lambda: mma.mma_kv_offload(xlay, pool, layers, src_blocks, plan.dest, stream), reps=5,
                    warm=1)
        extras[key] = {
            "fetch_ms": round(xf["p50"], 3), "fetch_GBs": round(total / xf["p50"] / 1e6, 2),
            "fetch_frac_of_measured": round(total / xf["p50"] / 1e6 / m_h2d, 4),
            "offload_2048_ms": round(xo["p50"], 3), "offload_GBs": round(off_bytes / xo["p50"] / 1e6, 2),
            "offload_frac_of_measured_d2h": round(off_bytes / xo["p50"] / 1e6 / m_d2h, 4),
            "sampled_parity": ok_x}
        log(key, extras[key])

    # Measured HBM copy peak (read + write bytes), 2 GiB each way: the best of the runtime's
    # device-to-device copy, the bare grid-stride streaming kernel and a span copy (whole 16 KiB
    # spans per wave, nontemporal), each streaming kernel at the best grid of a sweep.
    hb = 2 << 30
    ha = torch.empty(hb, dtype=torch.uint8, device="cuda")
    hbuf2 = torch.empty(hb, dtype=torch.uint8, device="cuda")
    with torch.cuda.stream(stream):
        d2d = _timed(stream, lambda: hbuf2.copy_(ha), reps=5, warm=1)["p50"]
    cs = ctypes.c_void_p(stream.cuda_stream)
    grids = (512, 1024, 2048, 4096, 8192, 16384)
    zc = {g: _timed(stream, lambda: nat.native_zero_copy(hbuf2.data_ptr(), ha.data_ptr(), hb, 0, g, cs), reps=5,
                    warm=1)["p50"] for g in grids}
    sc = {g: _timed(stream, lambda: nat.native_hbm_copy(hbuf2.data_ptr(), ha.data_ptr(), hb, g, cs), reps=5,
                    warm=1)["p50"] for g in grids}
    gbest, sbest = min(zc, key=zc.get), min(sc, key=sc.get)
    hbm_peak = max(2 * hb / d2d / 1e6, 2 * hb / zc[gbest] / 1e6, 2 * hb / sc[sbest] / 1e6)
    extras["measured_hbm_copy"] = {"peak_GBs_read_plus_write": round(hbm_peak, 1),
                                   "device_copy_GBs": round(2 * hb / d2d / 1e6, 1),
                                   "streaming_kernel_GBs": round(2 * hb / zc[gbest] / 1e6, 1),
                                   "streaming_kernel_grid": gbest,
                                   "span_copy_kernel_GBs": round(2 * hb / sc[sbest] / 1e6, 1),
                                   "span_copy_kernel_grid": sbest, "theoretical_GBs": 8000.0}
    del ha, hbuf2

    # The same gather with the pool resident in HBM: the CU gather/scatter code alone, HBM-bound.
    r = np.random.default_rng(1)
    dpool = torch.empty(s.host_num_slots * s.slot_bytes, dtype=torch.uint8, device="cuda")
    dpool.copy_(torch.from_numpy(pool.array))
    hbm = _timed(stream, lambda: mma.mma_kv_fetch(lay, dpool, layers, hs, gb, stream), reps=5, warm=1)
    ok_hbm = True
    pv4 = pool.array.reshape(s.host_num_slots, s.layers, 2, -1)
    for _ in range(16):
        i, l, k = int(r.integers(s.n_blocks)), int(r.integers(s.layers)), int(r.integers(2))
        o = (k * s.gpu_num_blocks + int(gb[i])) * s.piece_bytes
        ok_hbm &= bool(np.array_equal(layers[l][o:o + s.piece_bytes].cpu().numpy(), pv4[hs[i], l, k]))
    extras["kv_gather_hbm_pool"] = {"ms": round(hbm["p50"], 3), "payload_GBs": round(total / hbm["p50"] / 1e6, 1),
                                    "hbm_GBs_read_plus_write": round(2 * total / hbm["p50"] / 1e6, 1),
                                    "frac_of_8TBs": round(2 * total / hbm["p50"] / 1e6 / 8000.0, 4),
                                    "frac_of_measured_copy": round(2 * total / hbm["p50"] / 1e6 / hbm_peak, 4),
                                    "sampled_parity": ok_hbm}
    del dpool

    # Model wake-up: 291 Llama-3-8B-shaped bf16 tensors (16.06 GB) as one list, against 291 hipMemcpyAsync.
    sizes = W.weight_tensor_bytes()
    offs, wtotal = W.arena_offsets(sizes, 256)
    arena = mma.PinnedBuffer(wtotal)
    arena.array[::4096] = 0x3C
    wdst = [torch.empty(k, dtype=torch.uint8, device="cuda") for k in sizes]
    lst = [(wdst[t], arena.ptr + offs[t], sizes[t]) for t in range(len(sizes))]
    w = _timed(stream, lambda: mma.mma_weights_load(lst, mma.MMA_H2D, stream), reps=3, warm=1)
    Dw = (ctypes.c_void_p * len(sizes))(*[t.data_ptr() for t in wdst])
    Sw = (ctypes.c_void_p * len(sizes))(*[arena.ptr + o for o in offs])
    Zw = (ctypes.c_uint64 * len(sizes))(*sizes)
    wn = _timed(stream, lambda: nat.native_list(Dw, Sw, Zw, len(sizes), 0, ctypes.c_void_p(stream.cuda_stream)),
                reps=3, warm=1)
    extras["weights_wakeup_291"] = {"mma_ms": round(w["p50"], 2), "mma_GBs": round(wtotal / w["p50"] / 1e6, 2),
                                    "native_ms": round(wn["p50"], 2), "ratio_vs_native": round(wn["p50"] / w["p50"], 3)}
    # The reverse ("fall asleep"): the same 291 tensors device -> host into the arena.
    back = [(arena.ptr + offs[t], wdst[t], sizes[t]) for t in range(len(sizes))]
    ws = _timed(stream, lambda: mma.mma_weights_load(back, mma.MMA_D2H, stream), reps=3, warm=1)
    wsn = _timed(stream, lambda: nat.native_list(Sw, Dw, Zw, len(sizes), 1, ctypes.c_void_p(stream.cuda_stream)),
                 reps=3, warm=1)
    extras["weights_sleep_291"] = {"mma_ms": round(ws["p50"], 2), "mma_GBs": round(wtotal / ws["p50"] / 1e6, 2),
                                   "native_ms": round(wsn["p50"], 2),
                                   "ratio_vs_native": round(wsn["p50"] / ws["p50"], 3)}

    # Mixed contention: the wake-up list as 34 groups on stream A, each followed by the dependent
    # digest kernel over the group, while the 2048-block offload runs on stream B; 256 KiB chunks.
    # A and B run side by side (see side_by_side_schedules).
    extras["mixed_contention"] = mixed_contention(mma, W, np, torch, s, nat, pool, layers, lay, src_blocks, plan,
                                                  arena, offs, sizes, wdst, Dw, Sw, Zw, lp)
    mc = extras["mixed_contention"]
    mc["duplex_probe_GBs"] = peaks.get("duplex_GBs")
    if mc["mma"].get("overlap_aggregate_GBs") and peaks.get("duplex_GBs"):
        mc["overlap_frac_of_duplex_probe"] = round(mc["mma"]["overlap_aggregate_GBs"] / peaks["duplex_GBs"], 3)

    # All five workloads under both control modes, with the engine threads' CPU time per call.
    extras["control_modes"] = control_modes(mma, W, np, torch, nat, s, pool, layers, lay, hs, gb, src_blocks, plan,
                                            arena, offs, sizes, wdst, Dw, Sw, Zw, lp)
    extras["device_control"] = extras["control_modes"]["device"]["kv_fetch_64k"]
    del wdst
    arena.free()
    return extras


def control_modes(mma, W, np, torch, nat, s, pool, layers, lay, hs, gb, src_blocks, plan, arena, offs, sizes, wdst,
                  Dw, Sw, Zw, lp):
    """The five workloads under host control (engine threads pull for every path) and device control
    (the calling thread plans each transfer, the dummy-task kernel alone tracks it), each on a
    stream of its own: median time and GB/s, and the engine threads' CPU time per call (their
    CPU-time delta over the timed calls, read after they have gone idle)."""
    import ctypes
    stream = torch.cuda.Stream()
    n64 = W.COPY64_BYTES
    src64 = mma.PinnedBuffer(n64)
    src64.array[:] = W.uniform_bytes(1, W.TAG_DATA, 0, n64)
    dst64 = torch.empty(n64, dtype=torch.uint8, device="cuda")
    wtotal = sum(sizes)
    lst = [(wdst[t], arena.ptr + offs[t], sizes[t]) for t in range(len(sizes))]
    off_bytes = len(src_blocks) * s.slot_bytes
    total = s.n_blocks * s.slot_bytes
    margs = (ctypes.c_void_p(dst64.data_ptr()), ctypes.c_void_p(src64.ptr), ctypes.c_uint64(n64), mma.MMA_H2D,
             ctypes.c_void_p(stream.cuda_stream))

    def cpu_ns():
        mma.mma_synchronize()
        time.sleep(0.005)  # past the engine threads' spin after their last transfer
        return mma.mma_get_stats()["engine_cpu_ns"]

    def leg(fn, reps, warm, nbytes):
        for _ in range(warm):
            fn()
        stream.synchronize()
        c0 = cpu_ns()
        t = _timed(stream, fn, reps=reps, warm=0)
        c1 = cpu_ns()
        return {"ms": round(t["p50"], 3), "GBs": round(nbytes / t["p50"] / 1e6, 2),
                "engine_cpu_ms_per_call": round((c1 - c0) / 1e6 / reps, 3)}

    out = {}
    cfg0 = mma.mma_get_config()
    mma.mma_finalize()
    try:
        for mode, code in (("host", mma.MMA_CONTROL_HOST), ("device", mma.MMA_CONTROL_DEVICE)):
            c = _default_config()
            c.control = code
            mma.mma_init(0, c)
            r = {"copy_64mib": leg(lambda: _ok(mma.lib.mma_memcpy_async(*margs)), 20, 3, n64),
                 "weights_wakeup_291": leg(lambda: mma.mma_weights_load(lst, mma.MMA_H2D, stream), 2, 1, wtotal),
                 "kv_fetch_64k": leg(lambda: mma.mma_kv_fetch(lay, pool, layers, hs, gb, stream), 3, 1, total),
                 "kv_offload_2048": leg(lambda: mma.mma_kv_offload(lay, pool, layers, src_blocks, plan.dest, stream),
                                        3, 1, off_bytes)}
            ok64 = bool(np.array_equal(dst64[:1 << 20].cpu().numpy(), src64.array[:1 << 20]))
            r["copy_64mib"]["sampled_parity"] = ok64
            r["kv_fetch_64k"]["sampled_parity"] = sampled_fetch_parity(
                s, pool.array.reshape(s.host_num_slots, s.slot_bytes), layers, hs, gb, lay.gpu_layout, samples=16,
                seed=3)
            r["failed_transfers"] = mma.mma_get_stats()["failed_transfers"]
            mma.mma_finalize()
            c.chunk_bytes = 256 << 10
            mma.mma_init(0, c)
            c0 = cpu_ns()
            mx, _, tried = side_by_side_schedules(mma, torch, nat, s, W, pool, layers, lay, src_blocks, plan,
                                                  arena, offs, sizes, wdst, Dw, Sw, Zw, lp)
            c1 = cpu_ns()
            r["mixed_contention"] = {**mx, "stream_pairs_tried": tried,
                                     "engine_cpu_ms_per_schedule": round((c1 - c0) / 1e6 / (4 * tried), 3)}
            r["failed_transfers"] += mma.mma_get_stats()["failed_transfers"]
            mma.mma_finalize()
            out[mode] = r
            log(f"control {mode}:", r)
    finally:
        mma.mma_init(0, cfg0)
    src64.free()
    return out


def sampled_fetch_parity(s, pv, layers, hs, gb, gpu_layout, samples=64, seed=0):
    """Random (block, layer, K/V) pieces of the GPU cache against the pool bytes they were
    fetched from: the piece itself (gpu_layout 0), its x-packed key [H][D/x][B][x] / value
    [H][D][B] arrangement (1), or its head-major [H][B][D] arrangement (2)."""
    import numpy as np
    r = np.random.default_rng(seed)
    ok = True
    B_, H_, D_, E_ = s.block_tokens, s.kv_heads, s.head_dim, s.elem_bytes
    for _ in range(samples):
        i, l, k = int(r.integers(s.n_blocks)), int(r.integers(s.layers)), int(r.integers(2))
        off = (k * s.gpu_num_blocks + int(gb[i])) * s.piece_bytes
        got = layers[l][off:off + s.piece_bytes].cpu().numpy()
        want = pv[hs[i]].reshape(s.layers, 2, s.piece_bytes)[l, k]
        if gpu_layout == 1:
            w = want.reshape(B_, H_, D_, E_)
            want = (w.reshape(B_, H_, D_ * E_ // 16, 16 // E_, E_).transpose(1, 2, 0, 3, 4) if k == 0
                    else w.transpose(1, 2, 0, 3)).reshape(-1)
        elif gpu_layout == 2:
            want = want.reshape(B_, H_, D_ * E_).transpose(1, 0, 2).reshape(-1)
        ok &= bool(np.array_equal(got, want))
    return ok


def mixed_contention(mma, W, np, torch, s, nat, pool, layers, lay, src_blocks, plan, arena, offs, sizes, wdst,
                     Dw, Sw, Zw, lp):
    groups = W.weight_groups()
    assert all(list(g) == list(range(g[0], g[0] + len(g))) for g in groups)
    res = {}
    cfg = mma.mma_get_config()
    mma.mma_finalize()
    c = _default_config()
    c.chunk_bytes = 256 << 10
    mma.mma_init(0, c)
    try:
        for t in range(len(sizes)):
            wdst[t].fill_(W.WEIGHT_POISON)
        r, streams, tried = side_by_side_schedules(mma, torch, nat, s, W, pool, layers, lay, src_blocks, plan, arena,
                                                   offs, sizes, wdst, Dw, Sw, Zw, lp)
        r["stream_pairs_tried"] = tried
        mma.mma_synchronize()
        g = np.random.default_rng(2)
        ok = True
        for t in [int(x) for x in g.integers(len(sizes), size=8)]:
            ok &= bool(np.array_equal(wdst[t][:65536].cpu().numpy(), arena.array[offs[t]:offs[t] + min(65536, sizes[t])]))
        wtotal, off_bytes = sum(sizes), len(src_blocks) * s.slot_bytes
        a_ms, b_ms = r["stream_a_weights_digests_ms"], r["stream_b_offload_ms"]
        # both directions over the offload's time: its bytes, plus the weight bytes moved meanwhile
        # at stream A's average rate (only while the two ran side by side)
        agg = (off_bytes + wtotal / a_ms * b_ms) / b_ms / 1e6 if r["concurrent"] and b_ms <= a_ms else None
        res["mma"] = {**r, "overlap_aggregate_GBs": round(agg, 1) if agg else None, "sampled_parity": ok,
                      "failed_transfers": mma.mma_get_stats()["failed_transfers"]}
    finally:
        mma.mma_finalize()
        mma.mma_init(0, cfg)
    res["native"], _, tried = side_by_side_schedules(mma, torch, nat, s, W, pool, layers, lay, src_blocks, plan,
                                                     arena, offs, sizes, wdst, Dw, Sw, Zw, lp, native=True)
    res["native"]["stream_pairs_tried"] = tried
    res["makespan_speedup_vs_native"] = round(res["native"]["makespan_ms"] / res["mma"]["makespan_ms"], 3)
    res["stream_a_ratio_vs_native"] = round(res["native"]["stream_a_weights_digests_ms"] /
                                            res["mma"]["stream_a_weights_digests_ms"], 3)
    res["chunk_bytes"] = 256 << 10
    return res


# ---------------------------------------------------------------- sweeps (--sweep NAME)
def _sweep_env():
    import torch

    import paper_2512_16056_amd as mma
    torch.cuda.set_device(0)
    return mma, torch, native_lib(), torch.cuda.Stream()


def _emit(**rec):
    print(json.dumps(rec), flush=True)


def sweep_sizes():
    """Bandwidth against transfer size, both directions, 1 KiB to 8 GiB (the paper's microbenchmark
    range): the default multipath configuration against one hipMemcpyAsync of the same buffers.
    Median of HIP-event-bracketed runs on the launch stream."""
    import ctypes
    mma, torch, nat, st = _sweep_env()
    mma.mma_init(0)
    top = 8 << 30
    h = mma.PinnedBuffer(top)
    h.array[::4096] = 1
    d = torch.empty(top, dtype=torch.uint8, device="cuda")
    for n in [1 << k for k in range(10, 34)]:
        reps = 50 if n <= (64 << 20) else (10 if n <= (1 << 30) else 3)
        row = {"bytes": n}
        for dr, name in ((0, "h2d"), (1, "d2h")):
            dst, src = (d.data_ptr(), h.ptr) if dr == 0 else (h.ptr, d.data_ptr())
            D, S, Z = (ctypes.c_void_p * 1)(dst), (ctypes.c_void_p * 1)(src), (ctypes.c_uint64 * 1)(n)
            sp = ctypes.c_void_p(st.cuda_stream)
            t_nat = _timed(st, lambda: nat.native_list(D, S, Z, 1, dr, sp), reps, 3)
            margs = (ctypes.c_void_p(dst), ctypes.c_void_p(src), ctypes.c_uint64(n), dr, sp)
            t_mma = _timed(st, lambda: _ok(mma.lib.mma_memcpy_async(*margs)), reps, 3)
            row[name] = {"mma_us": round(t_mma["p50"] * 1e3, 2), "native_us": round(t_nat["p50"] * 1e3, 2),
                         "mma_GBs": round(n / t_mma["p50"] / 1e6, 2), "native_GBs": round(n / t_nat["p50"] / 1e6, 2),
                         "ratio_vs_native": round(t_nat["p50"] / t_mma["p50"], 3)}
        _emit(sweep="sizes", **row)
    h.free()
    mma.mma_finalize()


def sweep_misaligned():
    """Copies whose two ends differ in alignment modulo 16 (source at +1, destination at +0, and the
    reverse), 64 KiB to 64 MiB, both directions: the default multipath configuration against the
    same copy with both ends aligned and against one hipMemcpyAsync of the misaligned buffers.
    Median of HIP-event-bracketed runs on the launch stream."""
    import ctypes
    mma, torch, nat, st = _sweep_env()
    mma.mma_init(0)
    top = (64 << 20) + 64
    h = mma.PinnedBuffer(top)
    h.array[::4096] = 1
    d = torch.empty(top, dtype=torch.uint8, device="cuda")
    sp = ctypes.c_void_p(st.cuda_stream)
    for n in [1 << k for k in range(16, 27)]:
        reps = 30 if n <= (16 << 20) else 10
        row = {"bytes": n}
        for dr, name in ((0, "h2d"), (1, "d2h")):
            res = {}
            for tag, (so, do) in (("aligned", (0, 0)), ("src+1", (1, 0)), ("dst+1", (0, 1)), ("src+5,dst+9", (5, 9))):
                hp, dp = (h.ptr + so, d.data_ptr() + do) if dr == 0 else (h.ptr + do, d.data_ptr() + so)
                dst, src = (dp, hp) if dr == 0 else (hp, dp)
                margs = (ctypes.c_void_p(dst), ctypes.c_void_p(src), ctypes.c_uint64(n), dr, sp)
                t_mma = _timed(st, lambda: _ok(mma.lib.mma_memcpy_async(*margs)), reps, 3)
                ent = {"mma_us": round(t_mma["p50"] * 1e3, 2), "mma_GBs": round(n / t_mma["p50"] / 1e6, 2)}
                if tag != "aligned":
                    D, S, Z = (ctypes.c_void_p * 1)(dst), (ctypes.c_void_p * 1)(src), (ctypes.c_uint64 * 1)(n)
                    t_nat = _timed(st, lambda: nat.native_list(D, S, Z, 1, dr, sp), reps, 3)
                    ent["native_us"] = round(t_nat["p50"] * 1e3, 2)
                    ent["ratio_vs_native"] = round(t_nat["p50"] / t_mma["p50"], 3)
                    ent["ratio_vs_aligned"] = round(res["aligned"]["mma_us"] / ent["mma_us"], 3)
                res[tag] = ent
            row[name] = res
        _emit(sweep="misaligned", **row)
    h.free()
    mma.mma_finalize()


def sweep_idle(sizes=None):
    """Host wall time from the call to the return of hipStreamSynchronize, on a stream with nothing
    pending (the case of the idle-stream early start), for the default multipath configuration and
    one hipMemcpyAsync, alternating; the median after discarded warm-up calls (50 of 60 up to
    64 MiB, fewer above). Also the share of transfers whose copy engines started before the
    kernel's start signal (trace: started < 3 us after submission)."""
    import ctypes
    import numpy as np
    mma, torch, nat, st = _sweep_env()
    mma.mma_init(0)
    sizes = sizes or [32 << 10, 64 << 10, 256 << 10, 1 << 20, 4 << 20, 8 << 20, 16 << 20, 32 << 20, 64 << 20,
                      256 << 20, 1 << 30, 8 << 30]
    top = max(sizes)
    h = mma.PinnedBuffer(top)
    h.array[::4096] = 1
    d = torch.empty(top, dtype=torch.uint8, device="cuda")
    sp = ctypes.c_void_p(st.cuda_stream)
    # The platform's own round trips on an idle stream: a one-workgroup kernel (the digest kernel over
    # 4 bytes) and a 4-byte hipMemcpyAsync, each from the call to the return of hipStreamSynchronize.
    out8 = torch.zeros(1, dtype=torch.int64, device="cuda")
    D4, S4, Z4 = (ctypes.c_void_p * 1)(d.data_ptr()), (ctypes.c_void_p * 1)(h.ptr), (ctypes.c_uint64 * 1)(4)
    tk, tc = [], []
    for _ in range(60):
        st.synchronize()
        t0 = time.perf_counter()
        _ok(mma.lib.mma_digest_u32(ctypes.c_void_p(d.data_ptr()), ctypes.c_uint64(4), ctypes.c_void_p(out8.data_ptr()),
                                   sp))
        st.synchronize()
        tk.append((time.perf_counter() - t0) * 1e6)
        t0 = time.perf_counter()
        nat.native_list(D4, S4, Z4, 1, 0, sp)
        st.synchronize()
        tc.append((time.perf_counter() - t0) * 1e6)
    _emit(sweep="idle", reference="round trips of the platform, idle stream",
          tiny_kernel_us=round(float(np.median(tk[10:])), 1), tiny_copy_us=round(float(np.median(tc[10:])), 1))
    for n in sizes:
        reps, skip = (60, 10) if n <= (64 << 20) else ((14, 4) if n <= (1 << 30) else (5, 1))
        row = {"bytes": n}
        for dr, name in ((0, "h2d"), (1, "d2h")):
            dst, src = (d.data_ptr(), h.ptr) if dr == 0 else (h.ptr, d.data_ptr())
            D, S, Z = (ctypes.c_void_p * 1)(dst), (ctypes.c_void_p * 1)(src), (ctypes.c_uint64 * 1)(n)
            margs = (ctypes.c_void_p(dst), ctypes.c_void_p(src), ctypes.c_uint64(n), dr, sp)
            tn, tm, an, am = [], [], [], []
            mma.mma_trace_enable(True)
            for _ in range(reps):
                st.synchronize()
                t0 = time.perf_counter()
                nat.native_list(D, S, Z, 1, dr, sp)
                t1 = time.perf_counter()
                st.synchronize()
                tn.append((time.perf_counter() - t0) * 1e6)
                an.append((t1 - t0) * 1e6)
                time.sleep(0.0002)
                t0 = time.perf_counter()
                _ok(mma.lib.mma_memcpy_async(*margs))
                t1 = time.perf_counter()
                st.synchronize()
                tm.append((time.perf_counter() - t0) * 1e6)
                am.append((t1 - t0) * 1e6)
            mma.mma_synchronize()
            tr = mma.mma_trace_read()[-reps:]
            mma.mma_trace_enable(False)
            early = sum(1 for r in tr if r["t_started_ns"] and r["t_started_ns"] - r["t_submit_ns"] < 3000)
            m, nt = float(np.median(tm[skip:])), float(np.median(tn[skip:]))
            row[name] = {"mma_us": round(m, 1), "native_us": round(nt, 1), "ratio_vs_native": round(nt / m, 3),
                         "mma_call_us": round(float(np.median(am[skip:])), 1),
                         "native_call_us": round(float(np.median(an[skip:])), 1),
                         "early_start_frac": round(early / max(1, len(tr)), 2)}
        _emit(sweep="idle", **row)
    h.free()
    mma.mma_finalize()


def sweep_blocking(sizes=None):
    """Blocking copies on a stream with nothing pending: host wall time from the call to its return,
    median of the last 30 of 40 calls, alternating one hipMemcpyAsync + hipStreamSynchronize
    (native), mma_memcpy_async + hipStreamSynchronize, and the blocking mma_memcpy_stream. Run for
    the default configuration ("default") and with every copy kept off the whole-launch route
    ("engine": cu_whole_bytes[_d2h] = 1). From the trace of the asynchronous calls, for transfers
    the engine thread drives: when it published `complete` and when it retired the transfer,
    counted from the call."""
    import ctypes
    import numpy as np
    mma, torch, nat, st = _sweep_env()
    sizes = sizes or [64 << 10, 256 << 10, 1 << 20, 4 << 20, 8 << 20, 16 << 20, 64 << 20]
    top = max(sizes)
    for mode in ("default", "engine"):
        cfg = _default_config()
        if mode == "engine":
            cfg.cu_whole_bytes = cfg.cu_whole_bytes_d2h = 1
        mma.mma_init(0, cfg)
        h = mma.PinnedBuffer(top)
        h.array[::4096] = 1
        d = torch.empty(top, dtype=torch.uint8, device="cuda")
        sp = ctypes.c_void_p(st.cuda_stream)
        outcome = ctypes.c_int32(0)
        for n in sizes:
            row = {"mode": mode, "bytes": n}
            for dr, name in ((0, "h2d"), (1, "d2h")):
                dst, src = (d.data_ptr(), h.ptr) if dr == 0 else (h.ptr, d.data_ptr())
                D, S, Z = (ctypes.c_void_p * 1)(dst), (ctypes.c_void_p * 1)(src), (ctypes.c_uint64 * 1)(n)
                margs = (ctypes.c_void_p(dst), ctypes.c_void_p(src), ctypes.c_uint64(n), dr, sp)
                tn, ta, tb, starts = [], [], [], []
                mma.mma_trace_enable(True)
                for _ in range(40):
                    st.synchronize()
                    t0 = time.perf_counter_ns()
                    nat.native_list(D, S, Z, 1, dr, sp)
                    st.synchronize()
                    tn.append(time.perf_counter_ns() - t0)
                    time.sleep(0.0002)
                    t0 = time.perf_counter_ns()
                    _ok(mma.lib.mma_memcpy_async(*margs))
                    st.synchronize()
                    ta.append(time.perf_counter_ns() - t0)
                    starts.append(t0)
                    mma.mma_synchronize()
                    time.sleep(0.0002)
                    t0 = time.perf_counter_ns()
                    _ok(mma.lib.mma_memcpy_stream(*margs, ctypes.byref(outcome)))
                    tb.append(time.perf_counter_ns() - t0)
                    time.sleep(0.0002)
                mma.mma_synchronize()
                recs = mma.mma_trace_read()[-80:][0::2]  # the asynchronous calls' records
                mma.mma_trace_enable(False)
                got = mma.mma_get_config()
                limit = got.cu_whole_bytes if dr == 0 else got.cu_whole_bytes_d2h
                eng = list(zip(recs, starts))[10:] if n > limit else []  # engine-driven transfers only
                med = lambda v: round(float(np.median(v[10:])) / 1e3, 1)
                row[name] = {"native_us": med(tn), "async_sync_us": med(ta), "blocking_us": med(tb),
                             "complete_us": round(float(np.median([(r["t_complete_ns"] - t) / 1e3 for r, t in eng])), 1)
                             if eng else None,
                             "retire_us": round(float(np.median([(r["t_retire_ns"] - t) / 1e3 for r, t in eng])), 1)
                             if eng else None}
            _emit(sweep="blocking", **row)
        h.free()
        mma.mma_finalize()


def _busy_timed(torch, st, fn, reps, warm):
    """HIP-event time of fn() queued behind about a millisecond of other work on `st`: the
    stream has work pending when fn is called. Median and the list, in ms."""
    ts = []
    for i in range(reps + warm):
        with torch.cuda.stream(st):
            torch.cuda._sleep(2_000_000)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(st)
        fn()
        e1.record(st)
        e1.synchronize()
        if i >= warm:
            ts.append(e0.elapsed_time(e1))
    ts.sort()
    return ts[len(ts) // 2]


def sweep_control():
    """Host control (the direction's engine thread pulls micro-tasks for every path) against
    device control (the calling thread plans the whole transfer, the dummy-task kernel alone
    tracks completion), on the same copies, both directions. Per mode:
      idle_us   host wall time from the call to the return of hipStreamSynchronize on a stream
                with nothing pending (both modes use the copy engines), median;
      api_us    time spent inside the call itself on that idle stream, median;
      busy_GBs  HIP-event rate of the copy queued behind other work on its stream (device
                control: the CU path alone);
      engine_cpu_us_per_transfer  CPU time of the engine threads over both legs / transfers.
    Then device control's CU-path share (static_cu_percent) on 1 GiB idle-stream copies."""
    import ctypes
    import numpy as np
    mma, torch, nat, st = _sweep_env()
    top = 1 << 30
    sp = ctypes.c_void_p(st.cuda_stream)
    sizes = [64 << 10, 1 << 20, 4 << 20, 16 << 20, 64 << 20, 256 << 20, 1 << 30]

    def idle_leg(margs, reps, warm):
        tw, ta = [], []
        for i in range(reps + warm):
            st.synchronize()
            t0 = time.perf_counter()
            _ok(mma.lib.mma_memcpy_async(*margs))
            t1 = time.perf_counter()
            st.synchronize()
            t2 = time.perf_counter()
            if i >= warm:
                tw.append((t2 - t0) * 1e6)
                ta.append((t1 - t0) * 1e6)
        return float(np.median(tw)), float(np.median(ta))

    rows = {}
    for mode, name in ((mma.MMA_CONTROL_HOST, "host"), (mma.MMA_CONTROL_DEVICE, "device")):
        cfg = _default_config()
        cfg.control = mode
        mma.mma_init(0, cfg)
        h = mma.PinnedBuffer(top)
        h.array[::4096] = 1
        d = torch.empty(top, dtype=torch.uint8, device="cuda")
        for n in sizes:
            reps = 30 if n <= (64 << 20) else 8
            for dr, dname in ((0, "h2d"), (1, "d2h")):
                dst, src = (d.data_ptr(), h.ptr) if dr == 0 else (h.ptr, d.data_ptr())
                margs = (ctypes.c_void_p(dst), ctypes.c_void_p(src), ctypes.c_uint64(n), dr, sp)
                mma.mma_synchronize()
                cpu0 = mma.mma_get_stats()["engine_cpu_ns"]
                idle_us, api_us = idle_leg(margs, reps, 3)
                busy_ms = _busy_timed(torch, st, lambda: _ok(mma.lib.mma_memcpy_async(*margs)), reps, 2)
                mma.mma_synchronize()
                cpu1 = mma.mma_get_stats()["engine_cpu_ns"]
                rows.setdefault((n, dname), {})[name] = {
                    "idle_us": round(idle_us, 1), "idle_GBs": round(n / idle_us / 1e3, 2),
                    "api_us": round(api_us, 2), "busy_GBs": round(n / busy_ms / 1e6, 2),
                    "engine_cpu_us_per_transfer": round((cpu1 - cpu0) / 1e3 / (2 * reps + 5), 1)}
        h.free()
        del d
        mma.mma_finalize()
    for (n, dname), r in rows.items():
        _emit(sweep="control", bytes=n, dir=dname, **r)

    for pct in (40, 50, 60, 70, 80, 100):
        cfg = _default_config()
        cfg.control = mma.MMA_CONTROL_DEVICE
        cfg.static_cu_percent = pct
        mma.mma_init(0, cfg)
        h = mma.PinnedBuffer(top)
        h.array[::4096] = 1
        d = torch.empty(top, dtype=torch.uint8, device="cuda")
        row = {"cu_percent": pct}
        for dr, dname in ((0, "h2d"), (1, "d2h")):
            dst, src = (d.data_ptr(), h.ptr) if dr == 0 else (h.ptr, d.data_ptr())
            margs = (ctypes.c_void_p(dst), ctypes.c_void_p(src), ctypes.c_uint64(top), dr, sp)
            idle_us, _ = idle_leg(margs, 8, 2)
            row[dname + "_GBs"] = round(top / idle_us / 1e3, 2)
        h.free()
        del d
        mma.mma_finalize()
        _emit(sweep="control_cu_share", **row)


def sweep_chunks():
    """Chunk size x outstanding-queue depth on a 512 MiB copy (the paper's sensitivity study,
    Section 5.3): H2D and D2H GB/s, default path set."""
    mma, torch, nat, st = _sweep_env()
    n = 512 << 20
    mma.mma_init(0)
    h = mma.PinnedBuffer(n)
    h.array[::4096] = 1
    d = torch.empty(n, dtype=torch.uint8, device="cuda")
    mma.mma_finalize()
    for chunk in (256 << 10, 512 << 10, 1 << 20, 2 << 20, 4 << 20, 8 << 20, 16 << 20):
        for depth in (1, 2, 4):
            c = _default_config()
            c.chunk_bytes, c.queue_depth = chunk, depth
            mma.mma_init(0, c)
            r = {}
            for dr, name in ((0, "h2d"), (1, "d2h")):
                dst, src = (d, h) if dr == 0 else (h, d)
                t = _timed(st, lambda: mma.mma_memcpy_async(dst, src, n, dr, st), 8, 2)["p50"]
                r[name + "_GBs"] = round(n / t / 1e6, 2)
            mma.mma_finalize()
            _emit(sweep="chunks", bytes=n, chunk=chunk, queue_depth=depth, **r)
    h.free()


def sweep_contention():
    """Pull-based path selection against fixed CU:SDMA splits decided at plan time (the paper's
    static-split comparison, Section 5.1.2) on a 1024-block KV fetch (2 GiB), with background load
    on another stream: none, bf16 GEMMs on every CU, HBM-bound device copies, or competing native
    host->GPU copies on the same link. Median of 3."""
    import workloads as W
    mma, torch, nat, ts = _sweep_env()
    s = W.KV64K
    nblk = 1024
    hs, gb = W.kv_fetch_tables(s, cfg=3)
    hs, gb = hs[:nblk], gb[:nblk]
    mma.mma_init(0)
    pool = mma.PinnedBuffer(s.host_num_slots * s.slot_bytes)
    pool.array[::4096] = 7
    mma.mma_finalize()
    layers = [torch.empty(s.layer_bytes, dtype=torch.uint8, device="cuda") for _ in range(s.layers)]
    lay = mma.kv_layout(s.layers, s.block_tokens, s.kv_heads, s.head_dim, s.elem_bytes, s.gpu_num_blocks,
                        s.host_num_slots)
    bs = torch.cuda.Stream()
    A = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    B = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    C = torch.empty(8192, 8192, device="cuda", dtype=torch.bfloat16)
    H = torch.empty(1 << 30, dtype=torch.uint8).pin_memory()
    Dv = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    X = torch.empty(2 << 30, dtype=torch.uint8, device="cuda")
    Y = torch.empty(2 << 30, dtype=torch.uint8, device="cuda")

    def background(kind):
        with torch.cuda.stream(bs):
            if kind == "gemm":
                for _ in range(300):
                    torch.matmul(A, B, out=C)
            elif kind == "native_h2d":
                for _ in range(12):
                    Dv.copy_(H, non_blocking=True)
            elif kind == "hbm":
                for _ in range(60):
                    X.copy_(Y)

    CU = mma.MMA_PATH_CU
    policies = [("pull", {}), ("static_cu0", dict(path_mask_h2d=0x3)),
                ("static_cu33", dict(static_split=1, static_cu_percent=33)),
                ("static_cu50", dict(static_split=1, static_cu_percent=50)),
                ("static_cu67", dict(static_split=1, static_cu_percent=67)),
                ("static_cu100", dict(path_mask_h2d=CU))]
    for kind in ("none", "gemm", "hbm", "native_h2d"):
        for policy, kv in policies:
            c = _default_config()
            for k, v in kv.items():
                setattr(c, k, v)
            mma.mma_init(0, c)
            mma.mma_kv_fetch(lay, pool, layers, hs, gb, ts)
            torch.cuda.synchronize()
            res = []
            for _ in range(3):
                mma.mma_reset_stats()
                background(kind)
                time.sleep(0.003)
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record(ts)
                mma.mma_kv_fetch(lay, pool, layers, hs, gb, ts)
                b.record(ts)
                torch.cuda.synchronize()
                mma.mma_synchronize()
                stt = mma.mma_get_stats()
                res.append((a.elapsed_time(b), stt["path_bytes"][16], sum(stt["path_bytes"][:16]), stt))
            mma.mma_finalize()
            res.sort(key=lambda x: x[0])
            ms, cu, sd, stt = res[1]
            _emit(sweep="contention", background=kind, policy=policy, ms=round(ms, 2),
                  GBs=round(nblk * s.slot_bytes / ms / 1e6, 2), cu_share=round(cu / max(1, cu + sd), 3),
                  foreign_skips=stt["sdma_foreign_busy_skips"], backoffs=stt["sdma_congestion_backoffs"])
    pool.free()


def sweep_duplex():
    """Both directions at once on one link: 1 GiB each way with raw probes (one hipMemcpyAsync per
    direction, one SDMA engine per direction, zero-copy kernels), then a 2 GiB KV fetch concurrent
    with a 2 GiB KV offload through the multipath path."""
    import ctypes
    import threading

    import numpy as np

    import workloads as W
    mma, torch, nat, sa = _sweep_env()
    sb = torch.cuda.Stream()
    mma.mma_init(0)
    n = 1 << 30
    h1, h2 = mma.PinnedBuffer(n), mma.PinnedBuffer(n)
    d1 = torch.empty(n, dtype=torch.uint8, device="cuda")
    d2 = torch.empty(n, dtype=torch.uint8, device="cuda")

    def both(fa, fb, nbytes_a, nbytes_b, reps=3):
        out = []
        for _ in range(reps + 1):
            torch.cuda.synchronize()
            ea = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            eb = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ea[0].record(sa)
            eb[0].record(sb)
            fa()
            ea[1].record(sa)
            fb()
            eb[1].record(sb)
            torch.cuda.synchronize()
            out.append((ea[0].elapsed_time(ea[1]), eb[0].elapsed_time(eb[1])))
        a = sorted(x[0] for x in out[1:])[reps // 2]
        b = sorted(x[1] for x in out[1:])[reps // 2]
        return {"h2d_ms": round(a, 3), "d2h_ms": round(b, 3),
                "aggregate_GBs": round(nbytes_a / a / 1e6 + nbytes_b / b / 1e6, 2)}

    D1, S1, Z = (ctypes.c_void_p * 1)(d1.data_ptr()), (ctypes.c_void_p * 1)(h1.ptr), (ctypes.c_uint64 * 1)(n)
    D2, S2 = (ctypes.c_void_p * 1)(h2.ptr), (ctypes.c_void_p * 1)(d2.data_ptr())
    _emit(sweep="duplex", case="hipMemcpyAsync h2d || d2h",
          **both(lambda: nat.native_list(D1, S1, Z, 1, 0, ctypes.c_void_p(sa.cuda_stream)),
                 lambda: nat.native_list(D2, S2, Z, 1, 1, ctypes.c_void_p(sb.cuda_stream)), n, n))
    _emit(sweep="duplex", case="zero-copy kernel h2d || d2h (64 WGs each)",
          **both(lambda: nat.native_zero_copy(d1.data_ptr(), h1.ptr, n, 0, 64, ctypes.c_void_p(sa.cuda_stream)),
                 lambda: nat.native_zero_copy(h2.ptr, d2.data_ptr(), n, 1, 64, ctypes.c_void_p(sb.cuda_stream)),
                 n, n))
    res = []
    for _ in range(4):
        ns = [ctypes.c_uint64(0), ctypes.c_uint64(0)]
        th = [threading.Thread(target=lambda: nat.native_sdma_all(d1.data_ptr(), h1.ptr, n, 0, 1, 0,
                                                                  ctypes.byref(ns[0]))),
              threading.Thread(target=lambda: nat.native_sdma_all(h2.ptr, d2.data_ptr(), n, 1, 2, 0,
                                                                  ctypes.byref(ns[1])))]
        for t in th:
            t.start()
        for t in th:
            t.join()
        res.append((ns[0].value / 1e6, ns[1].value / 1e6))
    a = sorted(x[0] for x in res[1:])[1]
    b = sorted(x[1] for x in res[1:])[1]
    _emit(sweep="duplex", case="SDMA engine 0 h2d || engine 1 d2h (host-timed)", h2d_ms=round(a, 3),
          d2h_ms=round(b, 3), aggregate_GBs=round(n / a / 1e6 + n / b / 1e6, 2))
    h1.free()
    h2.free()
    mma.mma_finalize()

    s = W.KV64K
    nb = 1024
    mma.mma_init(0)
    pool = mma.PinnedBuffer(s.host_num_slots * s.slot_bytes)
    mma.mma_finalize()
    layers = [torch.zeros(s.layer_bytes, dtype=torch.uint8, device="cuda") for _ in range(s.layers)]
    lay = mma.kv_layout(s.layers, s.block_tokens, s.kv_heads, s.head_dim, s.elem_bytes, s.gpu_num_blocks,
                        s.host_num_slots)
    hs, gb = W.kv_fetch_tables(s, cfg=3)
    hs1, gb1 = hs[:nb].astype(np.int32), gb[:nb].astype(np.int32)
    hs2, gb2 = hs[nb:2 * nb].astype(np.int32), gb[nb:2 * nb].astype(np.int32)
    kvb = nb * s.slot_bytes
    CU = mma.MMA_PATH_CU
    SAME = mma.MMA_DUPLEX_UNCHANGED
    for name, kv in (("default", {}),
                     ("all paths shared by both directions", dict(duplex_paths_h2d=SAME, duplex_paths_d2h=SAME)),
                     ("cu only", dict(path_mask_h2d=CU, path_mask_d2h=CU)),
                     ("d2h without cu", dict(path_mask_d2h=0x3)),
                     ("h2d without cu", dict(path_mask_h2d=0x3)),
                     ("no cu either way", dict(path_mask_h2d=0x3, path_mask_d2h=0x3)),
                     ("engine 0 h2d, engine 1 d2h, no cu", dict(path_mask_h2d=1, path_mask_d2h=2)),
                     ("engine 0 + cu h2d, engine 1 + cu d2h", dict(path_mask_h2d=CU | 1, path_mask_d2h=CU | 2)),
                     ("engine 0 h2d, engine 1 + cu d2h", dict(path_mask_h2d=1, path_mask_d2h=CU | 2))):
        c = _default_config()
        for k, v in kv.items():
            setattr(c, k, v)
        mma.mma_init(0, c)
        r = both(lambda: mma.mma_kv_fetch(lay, pool, layers, hs1, gb1, sa),
                 lambda: mma.mma_kv_offload(lay, pool, layers, gb2, hs2, sb), kvb, kvb)
        _emit(sweep="duplex", case=f"multipath kv fetch || kv offload: {name}", **r,
              failed=mma.mma_get_stats()["failed_transfers"])
        mma.mma_finalize()
    pool.free()


def sweep_mixed(sizes=None, rounds=6):
    """The mixed-contention workload (the 291-tensor list as 34 groups on stream A, each followed by
    the dependent digest kernel; the 2048-block KV offload on stream B; 256 KiB micro-tasks) under
    path assignments per direction, against the same schedule with native copies. The cases are
    interleaved over `rounds` rounds (a fresh library per run, one warm-up schedule, one timed), on
    one pair of streams shown to run side by side, and every run is reported: both streams' times,
    B's start, the makespan, and the link aggregate while both directions run (bytes of B plus the
    bytes A moved meanwhile at its average rate, over B's time)."""
    import ctypes

    import numpy as np

    import workloads as W
    mma, torch, nat, _ = _sweep_env()
    s = W.KV64K
    plan = W.kv_offload_plan(s, cfg=4)
    mma.mma_init(0)
    pool = mma.PinnedBuffer(s.host_num_slots * s.slot_bytes)
    pool.array[::4096] = 1
    sizes_w = W.weight_tensor_bytes()
    offs, wtotal = W.arena_offsets(sizes_w, 256)
    arena = mma.PinnedBuffer(wtotal)
    arena.array[::4096] = 0x3C
    mma.mma_finalize()
    layers = [torch.zeros(s.layer_bytes, dtype=torch.uint8, device="cuda") for _ in range(s.layers)]
    lay = mma.kv_layout(s.layers, s.block_tokens, s.kv_heads, s.head_dim, s.elem_bytes, s.gpu_num_blocks,
                        s.host_num_slots)
    hs, gb = W.kv_fetch_tables(s, cfg=3)
    src_blocks = gb[plan.dirty].astype(np.int32)
    off_bytes = len(plan.dirty) * s.slot_bytes
    wdst = [torch.empty(k, dtype=torch.uint8, device="cuda") for k in sizes_w]
    Dw = (ctypes.c_void_p * len(sizes_w))(*[t.data_ptr() for t in wdst])
    Sw = (ctypes.c_void_p * len(sizes_w))(*[arena.ptr + o for o in offs])
    Zw = (ctypes.c_uint64 * len(sizes_w))(*sizes_w)
    lp = (ctypes.c_void_p * s.layers)(*[t.data_ptr() for t in layers])
    CU = mma.MMA_PATH_CU
    SAME = mma.MMA_DUPLEX_UNCHANGED
    cases = [("default", {}),
             ("all paths shared by both directions", dict(duplex_paths_h2d=SAME, duplex_paths_d2h=SAME)),
             ("duplex h2d engines 0-1 + cu, d2h engines 2-5", dict(duplex_paths_h2d=CU | 0x3)),
             ("duplex h2d engines 0-1, d2h engines 2-3", dict(duplex_paths_d2h=0xC)),
             ("native", None)]
    c = _default_config()
    c.chunk_bytes = 256 << 10
    mma.mma_init(0, c)
    r, streams, tried = side_by_side_schedules(mma, torch, nat, s, W, pool, layers, lay, src_blocks, plan, arena,
                                               offs, sizes_w, wdst, Dw, Sw, Zw, lp, reps=1)
    mma.mma_finalize()
    _emit(sweep="mixed", streams_side_by_side=r["concurrent"], stream_pairs_tried=tried)
    for rnd in range(rounds):
        for name, kv in cases[rnd % len(cases):] + cases[:rnd % len(cases)]:
            c = _default_config()
            c.chunk_bytes = 256 << 10
            for k, v in (kv or {}).items():
                setattr(c, k, v)
            mma.mma_init(0, c)
            mma.mma_trace_enable(True)
            r = mixed_contention_schedules(mma, torch, nat, s, W, pool, layers, lay, src_blocks, plan, arena,
                                           offs, sizes_w, wdst, Dw, Sw, Zw, lp, native=kv is None, reps=1,
                                           streams=streams)
            a, b = r["stream_a_weights_digests_ms"], r["stream_b_offload_ms"]
            mma.mma_synchronize()
            st = mma.mma_get_stats()
            tr = mma.mma_trace_read()
            mma.mma_trace_enable(False)
            mma.mma_finalize()
            # micro-tasks per path of the timed schedule's transfers (the second half of the records)
            tr = tr[len(tr) // 2:]
            paths = {}
            for d, key in ((0, "h2d_tasks"), (1, "d2h_tasks")):
                tot = [0] * 17
                for r_ in tr:
                    if r_["dir"] == d:
                        tot = [x + y for x, y in zip(tot, r_["path_tasks"])]
                paths[key] = {("cu" if i == 16 else f"e{i}"): v for i, v in enumerate(tot) if v}
            agg = (off_bytes + wtotal / a * b) / b / 1e6 if r["concurrent"] and b <= a else None
            _emit(sweep="mixed", round=rnd, case=name, **r, overlap_aggregate_GBs=round(agg, 1) if agg else None,
                  failed=st["failed_transfers"], backoffs=st["sdma_congestion_backoffs"], **paths)
    arena.free()
    pool.free()


def side_by_side_schedules(mma, torch, nat, s, W, pool, layers, lay, src_blocks, plan, arena, offs, sizes, wdst,
                           Dw, Sw, Zw, lp, native=False, tries=6, reps=3):
    """mixed_contention_schedules on a pair of new streams that ran side by side. The runtime maps
    streams onto a few hardware queues (GPU_MAX_HW_QUEUES, 4 by default), and two streams may
    share one: a kernel or timing marker on one then waits for what was queued before it on the
    other, so the offload (and its first timing event) starts only when stream A has ended. The
    copy engines' commands of a runtime copy are ordered by stream, not by hardware queue, but
    the native schedule's timing events see the same wait. No separate probe predicts it (a sleep
    kernel on A beside an event or a kernel on B passed for pairs that then ran one after the
    other), so the schedule itself is the test: a pair whose offload started only after A ended
    is replaced by two new streams, up to `tries` times. Returns (result, streams, pairs tried)."""
    for k in range(tries):
        pair = (torch.cuda.Stream(), torch.cuda.Stream())
        r = mixed_contention_schedules(mma, torch, nat, s, W, pool, layers, lay, src_blocks, plan, arena, offs, sizes,
                                       wdst, Dw, Sw, Zw, lp, native=native, reps=reps, streams=pair)
        if r["concurrent"]:
            break
    return r, pair, k + 1


def mixed_contention_schedules(mma, torch, nat, s, W, pool, layers, lay, src_blocks, plan, arena, offs, sizes,
                               wdst, Dw, Sw, Zw, lp, native=False, reps=1, streams=None):
    """The mixed-contention schedule (stream A: 34 groups, each loaded and then digested; stream B:
    the offload, issued after A's work), once to warm up and then `reps` times. Medians in ms: A's
    and B's times on their streams, when B started after A's start, and the makespan from A's
    start to the later end; `concurrent`: B started before A ended in every timed run. `streams`:
    the (A, B) pair to use, else two new ones from torch's pool."""
    import ctypes
    groups = W.weight_groups()
    digests = torch.zeros(len(sizes), dtype=torch.int64, device="cuda")
    sa, sb = streams if streams else (torch.cuda.Stream(), torch.cuda.Stream())
    out = []
    for _ in range(reps + 1):
        ea = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        eb = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        torch.cuda.synchronize()
        t_host = time.perf_counter()
        ea[0].record(sa)
        for g in groups:
            if not native:
                mma.mma_weights_load([(wdst[t], arena.ptr + offs[t], sizes[t]) for t in g], mma.MMA_H2D, sa)
            else:
                o = 8 * g[0]
                nat.native_list(ctypes.addressof(Dw) + o, ctypes.addressof(Sw) + o, ctypes.addressof(Zw) + o,
                                len(g), 0, ctypes.c_void_p(sa.cuda_stream))
            for t in g:
                mma.mma_digest_u32(wdst[t], sizes[t], digests.data_ptr() + 8 * t, sa)
        ea[1].record(sa)
        b_host = (time.perf_counter() - t_host) * 1e3  # when the host got to issue B's work
        eb[0].record(sb)
        if not native:
            mma.mma_kv_offload(lay, pool, layers, src_blocks, plan.dest, sb)
        else:
            nat.native_kv_offload(pool.ptr, lp, src_blocks.ctypes.data_as(ctypes.c_void_p),
                                  plan.dest.ctypes.data_as(ctypes.c_void_p), len(src_blocks), s.layers,
                                  s.piece_bytes, s.gpu_num_blocks, ctypes.c_void_p(sb.cuda_stream))
        eb[1].record(sb)
        torch.cuda.synchronize()
        a, b, b0 = ea[0].elapsed_time(ea[1]), eb[0].elapsed_time(eb[1]), ea[0].elapsed_time(eb[0])
        out.append((a, b, b0, max(a, ea[0].elapsed_time(eb[1])), b_host))
    out = out[1:]

    def med(i):
        return sorted(x[i] for x in out)[len(out) // 2]
    return {"stream_a_weights_digests_ms": round(med(0), 1), "stream_b_offload_ms": round(med(1), 1),
            "stream_b_start_ms": round(med(2), 1), "makespan_ms": round(med(3), 1),
            "stream_b_issued_host_ms": round(med(4), 1), "concurrent": all(x[2] < x[0] for x in out)}


def sweep_paths():
    """Bandwidth against the path set (single-GPU analog of the paper's bandwidth-vs-paths study):
    a 1 GiB copy each way and a 1024-block (2 GiB) KV fetch with one engine, both host-facing
    engines, the CU path alone, and combinations; `all16` adds the xGMI-facing engines 2-15."""
    import workloads as W
    mma, torch, nat, st = _sweep_env()
    n = 1 << 30
    mma.mma_init(0)
    h = mma.PinnedBuffer(n)
    h.array[::4096] = 1
    s = W.KV64K
    pool = mma.PinnedBuffer(s.host_num_slots * s.slot_bytes)
    mma.mma_finalize()
    d = torch.empty(n, dtype=torch.uint8, device="cuda")
    layers = [torch.empty(s.layer_bytes, dtype=torch.uint8, device="cuda") for _ in range(s.layers)]
    lay = mma.kv_layout(s.layers, s.block_tokens, s.kv_heads, s.head_dim, s.elem_bytes, s.gpu_num_blocks,
                        s.host_num_slots)
    hs, gb = W.kv_fetch_tables(s, cfg=3)
    hs, gb = hs[:1024], gb[:1024]
    CU = mma.MMA_PATH_CU
    for name, mask in (("sdma0", 0x1), ("sdma1", 0x2), ("sdma0+1", 0x3), ("cu", CU), ("cu+sdma0", CU | 0x1),
                       ("cu+sdma0+1", CU | 0x3), ("cu+all16", CU | 0xFFFF)):
        c = _default_config()
        c.path_mask_h2d = c.path_mask_d2h = mask
        mma.mma_init(0, c)
        used = mma.mma_get_stats()
        r = {}
        for dr, nm in ((0, "h2d"), (1, "d2h")):
            dst, src = (d, h) if dr == 0 else (h, d)
            t = _timed(st, lambda: mma.mma_memcpy_async(dst, src, n, dr, st), 5, 1)["p50"]
            r[nm + "_GBs"] = round(n / t / 1e6, 2)
        t = _timed(st, lambda: mma.mma_kv_fetch(lay, pool, layers, hs, gb, st), 3, 1)["p50"]
        r["kv_fetch_GBs"] = round(1024 * s.slot_bytes / t / 1e6, 2)
        _emit(sweep="paths", paths=name, engines_h2d=hex(used["sdma_engines_h2d"]),
              cu=bool(used["cu_path_enabled"]), **r)
        mma.mma_finalize()
    h.free()
    pool.free()


def sweep_footprint():
    """Cost of the dummy task to other work on the GPU (the paper's claim that its spin kernel has
    a negligible footprint): 200 bf16 8192^3 matmuls alone, then next to back-to-back 1 GiB
    host->GPU copies: native hipMemcpyAsync, then multipath through the copy engines only (the dummy
    task is then a single waiting wave) and through the default path set (16 CU-path workgroups)."""
    mma, torch, nat, st = _sweep_env()
    n = 1 << 30
    mma.mma_init(0)
    h = mma.PinnedBuffer(n)
    mma.mma_finalize()
    d = torch.empty(n, dtype=torch.uint8, device="cuda")
    gs = torch.cuda.Stream()
    A = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    B = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    C = torch.empty(8192, 8192, device="cuda", dtype=torch.bfloat16)

    def gemms():
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        with torch.cuda.stream(gs):
            a.record(gs)
            for _ in range(200):
                torch.matmul(A, B, out=C)
            b.record(gs)
        return a, b

    torch.cuda.synchronize()
    gemms()
    torch.cuda.synchronize()
    a, b = gemms()
    torch.cuda.synchronize()
    alone = a.elapsed_time(b)
    _emit(sweep="footprint", case="gemm alone", gemm_ms=round(alone, 2))
    import ctypes
    mma.mma_init(0)
    D, S, Z = (ctypes.c_void_p * 1)(d.data_ptr()), (ctypes.c_void_p * 1)(h.ptr), (ctypes.c_uint64 * 1)(n)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(st)
    for _ in range(12):
        nat.native_list(D, S, Z, 1, 0, ctypes.c_void_p(st.cuda_stream))
    e1.record(st)
    a, b = gemms()
    torch.cuda.synchronize()
    g = a.elapsed_time(b)
    _emit(sweep="footprint", case="native hipMemcpyAsync copies (no dummy task)", gemm_ms=round(g, 2),
          gemm_slowdown=round(g / alone - 1, 4), copy_GBs=round(12 * n / e0.elapsed_time(e1) / 1e6, 2))
    mma.mma_finalize()
    # Reference points: one resident sleeping wave of any kernel, and a stream held by the command
    # processor (an event wait on a stream blocked in a host function): no wave resident.
    with torch.cuda.stream(st):
        torch.cuda._sleep(int(2.4e9 * 0.3))
    a, b = gemms()
    torch.cuda.synchronize()
    g = a.elapsed_time(b)
    _emit(sweep="footprint", case="one resident sleeping wave (torch.cuda._sleep)", gemm_ms=round(g, 2),
          gemm_slowdown=round(g / alone - 1, 4))
    hip = ctypes.CDLL("libamdhip64.so")
    cbt = ctypes.CFUNCTYPE(None, ctypes.c_void_p)
    hip.hipLaunchHostFunc.argtypes = [ctypes.c_void_p, cbt, ctypes.c_void_p]
    hold = cbt(lambda _: time.sleep(0.3))
    s3 = torch.cuda.Stream()
    hip.hipLaunchHostFunc(ctypes.c_void_p(s3.cuda_stream), hold, None)
    e3 = torch.cuda.Event()
    e3.record(s3)
    st.wait_event(e3)
    a, b = gemms()
    torch.cuda.synchronize()
    g = a.elapsed_time(b)
    _emit(sweep="footprint", case="stream held by the command processor (event wait, no wave)", gemm_ms=round(g, 2),
          gemm_slowdown=round(g / alone - 1, 4))
    # hipStreamWaitValue64 on signal memory (the documented form), released by a host store once the
    # matmuls are done: does the runtime hold the stream without a wave?
    vp, u64 = ctypes.c_void_p, ctypes.c_uint64
    hip.hipExtMallocWithFlags.argtypes = [ctypes.POINTER(vp), ctypes.c_size_t, ctypes.c_uint]
    hip.hipStreamWaitValue64.argtypes = [vp, vp, u64, ctypes.c_uint, u64]
    hip.hipStreamWriteValue64.argtypes = [vp, vp, u64, ctypes.c_uint]
    hip.hipStreamQuery.argtypes = [vp]
    hip.hipFree.argtypes = [vp]
    sig = vp()
    if hip.hipExtMallocWithFlags(ctypes.byref(sig), 8, 2) == 0:  # hipMallocSignalMemory
        val = ctypes.cast(sig, ctypes.POINTER(u64))
        torch.cuda.synchronize()
        val[0] = 0
        rc = hip.hipStreamWaitValue64(vp(st.cuda_stream), sig, 5, 0, (1 << 64) - 1)  # hipStreamWaitValueGte
        held = hip.hipStreamQuery(vp(st.cuda_stream)) != 0
        a, b = gemms()
        b.synchronize()
        g = a.elapsed_time(b)
        val[0] = 5
        t0 = time.perf_counter()
        while hip.hipStreamQuery(vp(st.cuda_stream)) != 0 and time.perf_counter() - t0 < 2.0:
            pass
        if hip.hipStreamQuery(vp(st.cuda_stream)) != 0:  # the store was not seen: the documented release
            hip.hipStreamWriteValue64(vp(s3.cuda_stream), sig, 6, 0)
        torch.cuda.synchronize()
        _emit(sweep="footprint", case="stream held by hipStreamWaitValue64 (signal memory)", wait_rc=rc,
              held=held, gemm_ms=round(g, 2), gemm_slowdown=round(g / alone - 1, 4),
              release_us=round((time.perf_counter() - t0) * 1e6, 1))
        hip.hipFree(sig)
    for name, mask in (("copy engines only (dummy task = 1 waiting wave)", 0x3),
                       ("default paths (16 CU-path workgroups)", 0)):
        c = _default_config()
        c.path_mask_h2d = mask
        mma.mma_init(0, c)
        mma.mma_memcpy_async(d, h, n, mma.MMA_H2D, st)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(st)
        for _ in range(12):
            mma.mma_memcpy_async(d, h, n, mma.MMA_H2D, st)
        e1.record(st)
        a, b = gemms()
        torch.cuda.synchronize()
        mma.mma_synchronize()
        g = a.elapsed_time(b)
        _emit(sweep="footprint", case=name, gemm_ms=round(g, 2), gemm_slowdown=round(g / alone - 1, 4),
              copy_GBs=round(12 * n / e0.elapsed_time(e1) / 1e6, 2),
              failed=mma.mma_get_stats()["failed_transfers"])
        mma.mma_finalize()
    h.free()

def sweep_hbmpool():
    """The 64k-token KV fetch (4096 blocks) and the 2048-block offload with the pool resident in HBM:
    one pool-kernel launch per call, GPU blocks in the piece and in the head-major layout. Reports
    HBM read+write TB/s per call (median of 5). After each direction, 32 sampled pieces are
    compared with the other side (for head-major blocks, through the [heads][tokens][row]
    permutation)."""
    import numpy as np

    import workloads as W
    mma, torch, nat, st = _sweep_env()
    s = W.KV64K
    hs, gb = W.kv_fetch_tables(s, cfg=3)
    plan = W.kv_offload_plan(s, cfg=4)
    mma.mma_init(0)
    torch.manual_seed(1)
    dpool = torch.empty(s.host_num_slots * s.slot_bytes, dtype=torch.uint8, device="cuda").random_(0, 256)
    layers = [torch.empty(s.layer_bytes, dtype=torch.uint8, device="cuda").random_(0, 256) for _ in range(s.layers)]
    lt = mma.layer_table(layers)
    torch.cuda.synchronize()
    r = np.random.default_rng(2)

    R = s.head_dim * s.elem_bytes

    def pieces_equal(slots, blocks, hnd):
        """32 sampled (slot, layer, K/V) pieces: the GPU block holds the pool piece, or for
        head-major blocks the piece's [tokens][heads][row] permuted to [heads][tokens][row]."""
        ok = True
        for _ in range(32):
            j, l, k = int(r.integers(len(slots))), int(r.integers(s.layers)), int(r.integers(2))
            po = int(slots[j]) * s.slot_bytes + (2 * l + k) * s.piece_bytes
            go = (k * s.gpu_num_blocks + int(blocks[j])) * s.piece_bytes
            piece, block = dpool[po:po + s.piece_bytes], layers[l][go:go + s.piece_bytes]
            if hnd:
                piece = piece.view(s.block_tokens, s.kv_heads, R).transpose(0, 1).contiguous().view(-1)
            ok &= bool(torch.equal(piece, block))
        return ok

    for name, code in (("piece", mma.MMA_KV_LAYOUT_PIECE), ("hnd", mma.MMA_KV_LAYOUT_HND)):
        lay = mma.kv_layout(s.layers, s.block_tokens, s.kv_heads, s.head_dim, s.elem_bytes, s.gpu_num_blocks,
                            s.host_num_slots, code)
        for case, fn, slots, blocks in (
                ("fetch", lambda: mma.mma_kv_fetch(lay, dpool, lt, hs, gb, st), hs, gb),
                ("offload", lambda: mma.mma_kv_offload(lay, dpool, lt, plan.src_blocks, plan.dest, st),
                 plan.dest, plan.src_blocks)):
            t = _timed(st, fn, reps=5, warm=1)
            st.synchronize()
            check = pieces_equal(slots, blocks, code == mma.MMA_KV_LAYOUT_HND)
            payload = len(slots) * s.slot_bytes
            _emit(sweep="hbmpool", layout=name, case=case, blocks=len(slots), payload_bytes=payload,
                  ms=round(t["p50"], 3), ms_p10_p90=[round(t["p10"], 3), round(t["p90"], 3)],
                  hbm_TBs_read_plus_write=round(2 * payload / t["p50"] / 1e9, 3),
                  frac_of_8TBs=round(2 * payload / t["p50"] / 1e9 / 8.0, 4),
                  check="32 sampled pieces against the other side", check_ok=check)
    mma.mma_finalize()


SWEEPS = {"sizes": sweep_sizes, "idle": sweep_idle, "chunks": sweep_chunks, "contention": sweep_contention, "duplex": sweep_duplex,
          "paths": sweep_paths, "footprint": sweep_footprint, "control": sweep_control, "hbmpool": sweep_hbmpool,
          "misaligned": sweep_misaligned, "mixed": sweep_mixed, "blocking": sweep_blocking}


def main():
    global _ENGINE_NAP_US
    args = parse()
    if args.engine_nap_us is not None:  # configurations built here, and mma_init without one
        _ENGINE_NAP_US = args.engine_nap_us
        os.environ["MMA_ENGINE_NAP_US"] = str(args.engine_nap_us)
    if args.control:
        os.environ["MMA_CONTROL"] = "1" if args.control == "device" else "0"
    if args.calib:
        calibration_kernels()
        return
    if args.oracle_cores:
        oracle_cores_worker([int(c) for c in args.oracle_cores.split(",")], args.cpu_seconds)
        return
    if args.sweep:
        if args.sizes:
            SWEEPS[args.sweep](sizes=[int(x, 0) for x in args.sizes.split(",")])
        else:
            SWEEPS[args.sweep]()
        return
    if args.gpus != 1:
        print(f"bench.py measures one GPU: the multipath path here is the single-GPU share (SDMA engines + "
              f"CU zero-copy over this GPU's own PCIe link); --gpus {args.gpus} is not supported.",
              file=sys.stderr)
        sys.exit(2)

    import ctypes

    import numpy as np

    import workloads as W

    s = W.KV64K
    hs, gb = W.kv_fetch_tables(s, cfg=3)
    total = s.n_blocks * s.slot_bytes
    # The batched native comparator runs as its own process, before this one touches the GPU.
    native_batch = None if args.no_extras else run_native_batch(s, hs, gb)
    log("native hipMemcpyBatchAsync:", native_batch)

    import torch

    import paper_2512_16056_amd as mma

    torch.cuda.set_device(0)

    mma.mma_init(0)  # defaults, then MMA_* environment overrides
    cfg = mma.mma_get_config().as_dict()
    log("config:", cfg)

    # ---- inputs: pinned 8 GiB pool (seeded, block i at host_slots[i]) and the GPU paged cache
    t0 = time.time()
    pool = mma.PinnedBuffer(s.host_num_slots * s.slot_bytes)
    pv = pool.array.reshape(s.host_num_slots, s.slot_bytes)

    def fill(i):
        pv[hs[i]] = W.kv_block_bytes(3, i, s)

    with ThreadPoolExecutor(16) as ex:
        list(ex.map(fill, range(s.n_blocks)))
    layers = [torch.full((s.layer_bytes,), W.GPU_POISON, dtype=torch.uint8, device="cuda") for _ in range(s.layers)]
    gl = {"piece": mma.MMA_KV_LAYOUT_PIECE, "xpacked": mma.MMA_KV_LAYOUT_XPACKED, "hnd": mma.MMA_KV_LAYOUT_HND}
    lay = mma.kv_layout(s.layers, s.block_tokens, s.kv_heads, s.head_dim, s.elem_bytes, s.gpu_num_blocks,
                        s.host_num_slots, gl[args.kv_layout])
    kernel_name = {"piece": "mma_transfer_kernel", "xpacked": "mma_transfer_xpacked_kernel",
                   "hnd": "mma_transfer_hnd_kernel"}[args.kv_layout]
    torch.cuda.synchronize()
    log(f"inputs ready in {time.time() - t0:.1f}s")

    stream = torch.cuda.Stream()
    for _ in range(args.warmup):
        mma.mma_kv_fetch(lay, pool, layers, hs, gb, stream)
    stream.synchronize()
    mma.mma_synchronize()
    mma.mma_reset_stats()

    # ---- timed region: exactly K steps, bracketed by synchronize on both sides
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    torch.cuda.synchronize()
    t_start = time.perf_counter()
    for a, b in ev:
        a.record(stream)
        mma.mma_kv_fetch(lay, pool, layers, hs, gb, stream)
        b.record(stream)
    torch.cuda.synchronize()
    t_end = time.perf_counter()
    elapsed = t_end - t_start
    mma.mma_synchronize()
    stats = mma.mma_get_stats()
    kernel_ms = [a.elapsed_time(b) for a, b in ev]
    avg_kernel_ms = sum(kernel_ms) / len(kernel_ms)
    kp = _pcts(kernel_ms)
    ms_per_step = elapsed * 1e3 / args.steps
    value = total * args.steps / elapsed / 1e9
    achieved = total / (avg_kernel_ms * 1e-3) / 1e9
    log(f"kv fetch: {ms_per_step:.2f} ms/step, {value:.2f} GB/s wall; kernel avg {avg_kernel_ms:.2f} ms "
        f"(min {min(kernel_ms):.2f}, max {max(kernel_ms):.2f}) = {achieved:.2f} GB/s")

    # ---- sampled parity against the definition of the fetch (full parity lives in the tests)
    ok = sampled_fetch_parity(s, pv, layers, hs, gb, lay.gpu_layout)
    log(f"sampled parity: {'ok' if ok else 'MISMATCH'}")

    # ---- host-observed latency: the call to the return of hipStreamSynchronize, stream idle
    host_ms = []
    for _ in range(5):
        stream.synchronize()
        t0 = time.perf_counter()
        mma.mma_kv_fetch(lay, pool, layers, hs, gb, stream)
        stream.synchronize()
        host_ms.append((time.perf_counter() - t0) * 1e3)
    hp = _pcts(host_ms)
    log(f"host-observed fetch latency: {hp['p50']:.3f} ms (p10 {hp['p10']:.3f}, p90 {hp['p90']:.3f})")

    out = {
        "metric": METRIC,
        "value": round(value, 3),
        "unit": "GB/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u8",
        "data": "synthetic",
        "config": {
            "workload": "kv_fetch_64k_tokens: 4096 blocks x 16 tokens, 32 layers x K,V x 8 kv heads x 128 dim bf16 "
                        "(8 GiB) pinned host pool -> paged GPU cache via block table"
                        + {"piece": "", "xpacked": " (x-packed GPU block layout)",
                           "hnd": " (head-major GPU block layout)"}[args.kv_layout],
            "gpu_block_layout": args.kv_layout,
            "bytes_per_step": total,
            "pieces_per_step": s.n_blocks * s.pieces_per_block,
            "chunk_bytes": cfg["chunk_bytes"],
            "paths_h2d": hex(cfg["path_mask_h2d"]),
            "cu_workgroups": cfg["cu_workgroups"],
            "control": "device" if cfg["control"] == mma.MMA_CONTROL_DEVICE else "host",
            "engine_nap_us": "off" if cfg["engine_nap_us"] == mma.MMA_ENGINE_NAP_OFF else cfg["engine_nap_us"],
            "parallelism": "1 GPU (SDMA engines + CU zero-copy on its own PCIe link)",
        },
        "kv_fetch_latency_ms": round(avg_kernel_ms, 3),
        "kv_fetch_latency_ms_p10_p50_p90": [round(kp[k], 3) for k in ("p10", "p50", "p90")],
        "kv_fetch_host_latency_ms": round(hp["p50"], 3),
        "kv_fetch_host_latency_ms_p10_p50_p90": [round(hp[k], 3) for k in ("p10", "p50", "p90")],
        "sampled_parity": ok,
        "path_bytes": {"cu": stats["path_bytes"][16],
                       **{f"sdma{e}": stats["path_bytes"][e] for e in range(16) if stats["path_bytes"][e]}},
        "engine_cpu_ms_per_step": round(stats["engine_cpu_ns"] / 1e6 / max(1, args.steps + args.warmup), 3),
        "engine_naps_per_step": round(stats["engine_naps"] / max(1, args.steps + args.warmup)),
        # SDMA share of the fetch: host slot -> HBM staging (copy engine), then the CU scatter
        # staging -> paged blocks reads and writes each byte once more in HBM.
        "staging_scatter": {
            "bytes_per_step": stats["staging_bytes"] // args.steps,
            "hbm_bytes_per_step": 2 * stats["staging_bytes"] // args.steps,
            "hbm_GBs_avg_over_step": round(2 * stats["staging_bytes"] / args.steps / (ms_per_step * 1e-3) / 1e9, 2),
            "frac_of_8TBs": round(2 * stats["staging_bytes"] / args.steps / (ms_per_step * 1e-3) / 8e12, 5),
        },
        "roofline": {
            "kernel": f"{kernel_name} (dummy task: CU gather + stream wait)",
            "bound": "pcie",
            "achieved": round(achieved, 3),
            "peak": round(PCIE5_X16_GBS, 2),
            "unit": "GB/s",
            "frac": round(achieved / PCIE5_X16_GBS, 4),
            "traffic": recorded_traffic(ROOT, kernel_name),
        },
    }

    extras = {}
    if not args.no_extras:
        extras = run_extras(mma, W, np, torch, s, pool, layers, lay, hs, gb, stream, ms_per_step, total, out,
                            native_batch)
        log("extras:", extras)
    out["extras"] = extras

    if not args.no_cpu_baseline:
        from oracle import kv as okv
        poison = np.full((2, s.gpu_num_blocks, s.piece_bytes), W.GPU_POISON, np.uint8)
        reps, t0 = 0, time.perf_counter()
        while True:
            for l in range(s.layers):
                okv.kv_fetch_layer(pv, poison, l, s.layers, hs, gb)
            reps += 1
            if time.perf_counter() - t0 >= args.cpu_seconds:
                break
        dt = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": round(total * reps / dt / 1e9, 3), "unit": "GB/s", "cores": 1,
                               "kind": "oracle",
                               "sample": f"{reps} x the full 4096-block 64k-token KV fetch (oracle.kv.kv_fetch_layer "
                                         f"over 32 layers, numpy slice copies, one thread), {dt:.1f} s"}
        # The same oracle over the cores near the GPU, one process per core, each on its own
        # disjoint slices of the block table: context for the host's own copy bandwidth. It runs
        # in a process of its own, which never touches the GPU (it forks its workers).
        out["cpu_baseline_all_cores"] = oracle_all_cores(torch, args.cpu_seconds / 2)
    print(json.dumps(out), flush=True)
    pool.free()
    mma.mma_finalize()


if __name__ == "__main__":
    main()

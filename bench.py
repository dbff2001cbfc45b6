#!/usr/bin/env python3
"""Benchmark of the AES-CTR hot path on one MI355X.

Workload (the headline): AES-128-CTR over 8 MiB buffers of uniform random
bytes, seeded key and nonce, counter from 1, inputs resident in HBM.  One
launch = one aes_ctr_crypt of one 8 MiB buffer (keystream + XOR, one kernel
launch).  One step = one replay of a captured HIP graph of K such launches
(K sized so a replay lasts at least 20 ms, recorded in
config.launches_per_step), so the replay's own fixed cost is spread over K
launches and the per-launch rate does not depend on --steps.  Buffers rotate
over more than 512 MiB so the 256 MB Infinity Cache cannot serve repeats.
The eager (one ctypes call per launch) rate is reported beside it.

Prints ONE JSON line.  Extra legs (the sweep with --sweep; the batch,
serving, hash and asyncio legs unless --no-batch / --no-serve / --no-hash /
--no-aio) add fields to that line; the CPU oracle leg (cpu_baseline) runs
unless --no-cpu.
"""
from __future__ import annotations

import argparse
import hashlib
import re
import json
import math
import os
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, HERE)

MiB = 1 << 20
HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, published


def log(msg: str) -> None:
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def parse():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20,
                    help="timed steps; a step is one replay of a captured graph of K launches")
    ap.add_argument("--warmup", type=int, default=5, help="untimed steps before the timed ones")
    ap.add_argument("--launches", type=int, default=0,
                    help="launches per step, K (0 = enough for a replay of at least 20 ms)")
    ap.add_argument("--size", type=int, default=8 * MiB, help="bytes per buffer")
    ap.add_argument("--bits", type=int, default=128, choices=(128, 256))
    ap.add_argument("--variant", type=int, default=0, help="0 auto, 1 T-table, 2 bitsliced, 3 vector permute")
    ap.add_argument("--sweep", action="store_true", help="also time 4 KiB..8 MiB + 256 MiB")
    ap.add_argument("--no-batch", action="store_true", help="skip the 4096-request batch leg")
    ap.add_argument("--no-serve", action="store_true", help="skip the serving-loop leg")
    ap.add_argument("--no-hash", action="store_true", help="skip the batched SHA-256 leg")
    ap.add_argument("--no-aio", action="store_true", help="skip the asyncio reroute leg")
    ap.add_argument("--serve-requests", type=int, default=100_000)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--cpu-seconds", type=float, default=10.0)
    return ap.parse_args()


class Timer:
    """HIP events on the stream the kernels run on (torch's current stream)."""

    def __init__(self, torch):
        self.torch = torch
        self.e0 = torch.cuda.Event(enable_timing=True)
        self.e1 = torch.cuda.Event(enable_timing=True)

    def __enter__(self):
        self.torch.cuda.synchronize()
        self.t0 = time.perf_counter()
        self.e0.record()
        return self

    def __exit__(self, *exc):
        self.e1.record()
        self.torch.cuda.synchronize()
        self.wall_ms = (time.perf_counter() - self.t0) * 1e3
        self.ms = self.e0.elapsed_time(self.e1)


def make_buffers(torch, W, size, bits, min_total=768 * MiB):
    payload = W.sweep_payload(size, bits)
    nbuf = max(2, math.ceil(min_total / (2 * size)))
    src = torch.from_numpy(payload).cuda()
    ins = [src.clone() for _ in range(nbuf)]
    outs = [torch.empty_like(src) for _ in range(nbuf)]
    return payload, ins, outs


def steady_state(torch, A, sched, nonce, ins, outs, steps, warmup, cfg=None, repeats=1):
    """K back-to-back launches replayed from one captured graph, timed over
    one replay (or the median of `repeats` replays)."""
    n = len(ins)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        for i in range(min(warmup, 3 * n)):
            A.aes_ctr_crypt(sched, nonce, 1, ins[i % n], outs[i % n], cfg=cfg)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for i in range(steps):
            A.aes_ctr_crypt(sched, nonce, 1, ins[i % n], outs[i % n], cfg=cfg)
    g.replay()                               # warm replays (clocks settle)
    g.replay()
    torch.cuda.synchronize()
    runs = []
    for _ in range(repeats):
        with Timer(torch) as t:
            g.replay()
        runs.append(t)
    runs.sort(key=lambda r: r.ms)
    return runs[len(runs) // 2], g


MIN_STEP_S = 0.020     # a timed step (one graph replay) lasts at least this long


def launches_for(torch, A, sched, nonce, ins, outs, cfg=None, min_s=MIN_STEP_S):
    """K, the launches per step: a graph of 100 launches is replayed three
    times and K is the smallest multiple of the buffer count whose replay
    lasts at least min_s at that rate."""
    n = len(ins)
    t, g = steady_state(torch, A, sched, nonce, ins, outs, 100, 0, cfg, repeats=3)
    del g
    per_launch_s = t.ms * 1e-3 / 100
    k = math.ceil(min_s / per_launch_s)
    return max(n, math.ceil(k / n) * n)


def replayed_steps(torch, A, sched, nonce, ins, outs, launches, steps, warmup, cfg=None):
    """The timed region: `steps` replays of one captured graph of `launches`
    back-to-back aes_ctr_crypt calls over the rotating buffers, after
    `warmup` untimed replays.  HIP events on the replay stream bracket the
    timed replays, with a device synchronisation on both sides.  Returns the
    Timer (ms = all timed steps)."""
    n = len(ins)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for i in range(launches):
            A.aes_ctr_crypt(sched, nonce, 1, ins[i % n], outs[i % n], cfg=cfg)
    for _ in range(max(warmup, 1)):
        g.replay()
    torch.cuda.synchronize()
    with Timer(torch) as t:
        for _ in range(steps):
            g.replay()
    del g
    return t


def eager(torch, A, sched, nonce, ins, outs, steps, cfg=None):
    n = len(ins)
    for i in range(min(steps, 20)):
        A.aes_ctr_crypt(sched, nonce, 1, ins[i % n], outs[i % n], cfg=cfg)
    with Timer(torch) as t:
        for i in range(steps):
            A.aes_ctr_crypt(sched, nonce, 1, ins[i % n], outs[i % n], cfg=cfg)
    return t


def single_latency_us(torch, A, sched, nonce, x, y, reps=50, cfg=None):
    vals = []
    for _ in range(reps):
        with Timer(torch) as t:
            A.aes_ctr_crypt(sched, nonce, 1, x, y, cfg=cfg)
        vals.append(t.ms * 1e3)
    vals.sort()
    return vals[len(vals) // 2]


def end_to_end_gbs(torch, A, sched, nonce, payload, reps=5):
    """Pinned host -> H2D -> kernel -> D2H on one stream."""
    n = len(payload)
    h_in = torch.from_numpy(payload).pin_memory()
    h_out = torch.empty(n, dtype=torch.uint8).pin_memory()
    d_in = torch.empty(n, dtype=torch.uint8, device="cuda")
    d_out = torch.empty_like(d_in)
    vals = []
    for _ in range(reps + 2):
        with Timer(torch) as t:
            d_in.copy_(h_in, non_blocking=True)
            A.aes_ctr_crypt(sched, nonce, 1, d_in, d_out)
            h_out.copy_(d_out, non_blocking=True)
        vals.append(n / (t.ms * 1e-3) / 1e9)
    vals = sorted(vals[2:])
    return vals[len(vals) // 2], h_out


def end_to_end_pipelined_gbs(torch, A, sched, nonce, payload, expect, chunk=1 * MiB, n_streams=2, reps=5):
    """Pinned host buffers, cut into chunks that go H2D -> kernel -> D2H on
    alternating streams, so one chunk's upload overlaps another's download
    (PCIe is full duplex).  Chunk i starts at counter 1 + i * chunk / 16."""
    n = len(payload)
    h_in = torch.from_numpy(payload).pin_memory()
    h_out = torch.empty(n, dtype=torch.uint8).pin_memory()
    d_in = torch.empty(n, dtype=torch.uint8, device="cuda")
    d_out = torch.empty_like(d_in)
    streams = [torch.cuda.Stream() for _ in range(n_streams)]
    cur = torch.cuda.current_stream()
    vals = []
    for _ in range(reps + 2):
        h_out.zero_()
        with Timer(torch) as t:
            for s in streams:
                s.wait_stream(cur)
            for i, off in enumerate(range(0, n, chunk)):
                m = min(chunk, n - off)
                s = streams[i % n_streams]
                with torch.cuda.stream(s):
                    d_in[off:off + m].copy_(h_in[off:off + m], non_blocking=True)
                    A.aes_ctr_crypt(sched, nonce, 1 + off // 16, d_in[off:off + m], d_out[off:off + m], stream=s)
                    h_out[off:off + m].copy_(d_out[off:off + m], non_blocking=True)
            for s in streams:
                cur.wait_stream(s)
        vals.append(n / (t.ms * 1e-3) / 1e9)
        if not torch.equal(h_out, expect):
            raise SystemExit("pipelined end-to-end output differs from the one-stream output")
    vals = sorted(vals[2:])
    return vals[len(vals) // 2]


def end_to_end_zero_copy_gbs(torch, A, sched, nonce, payload, expect, reps=5):
    """Pinned host buffers that the kernel reads and writes directly over
    PCIe: one request through the engine's host_buffers mode, timed on the
    host from submit to completion."""
    n = len(payload)
    h_in = torch.from_numpy(payload).pin_memory()
    h_out = torch.empty(n, dtype=torch.uint8).pin_memory()
    vals = []
    with A.Engine(n_streams=1, host_buffers=True) as eng:
        req = A.Request(sched, nonce, 1, h_in.data_ptr(), h_out.data_ptr(), n)
        for _ in range(reps + 8):
            h_out.zero_()
            t0 = time.perf_counter()
            eng.wait(eng.submit(req))
            vals.append(time.perf_counter() - t0)
            if not torch.equal(h_out, expect):
                raise SystemExit("zero-copy end-to-end output differs from the one-stream output")
    # The first passes over freshly pinned buffers run at a few GB/s on this
    # platform (several milliseconds per 8 MiB request, for up to about six
    # requests), and a new engine sets up its staging: eight untimed
    # requests, then the median of the rest.  Every request's time is
    # reported.
    timed = sorted(vals[8:])
    return n / timed[len(timed) // 2] / 1e9, [round(v * 1e6, 1) for v in vals]


TT_SOURCES = ("ttable_device.h", "ctr_ttable.hip", "aes_tables.h")


def kernel_source_hash() -> str:
    """sha256 of the T-table kernel's sources plus the text of the function
    that picks its default launch shape (so a host-side edit elsewhere does
    not void a counter summary, but a kernel or shape change does)."""
    csrc = os.path.join(HERE, "paper_2607_02630_amd", "csrc")
    h = hashlib.sha256()
    for name in TT_SOURCES:
        with open(os.path.join(csrc, name), "rb") as f:
            h.update(f.read())
    with open(os.path.join(csrc, "api.cpp")) as f:
        api = f.read()
    m = re.search(r"Shape default_shape\(.*?\n}\n", api, re.S)
    h.update(m.group(0).encode() if m else b"")
    # The tuner's entry for this workload overrides the rule where present.
    try:
        with open(os.path.join(HERE, "paper_2607_02630_amd", "tune_cache.json")) as f:
            entries = json.load(f).get("entries", [])
    except (OSError, ValueError):
        entries = []
    for e in entries:
        if (e.get("variant"), e.get("key_bits"), e.get("size_log2")) == (1, 128, 23):
            h.update(json.dumps(e, sort_keys=True).encode())
    return h.hexdigest()


def measured_traffic(bits, size, variant):
    """HBM bytes per launch from the committed rocprofv3 counter summary, if it
    was taken on this workload and on the kernel sources as they are now."""
    if (bits, size, variant) != (128, 8 * MiB, 0):
        return None
    path = os.path.join(HERE, "profiles", "ctr_ttable_aes128_8MiB_hbm_traffic.md")
    if not os.path.exists(path):
        return None
    fields = {}
    for line in open(path):
        if ":" in line and line.split(":")[0] in ("traffic_bytes_per_launch", "source_sha256"):
            k, v = line.split(":", 1)
            fields[k] = v.strip()
    if fields.get("source_sha256") != kernel_source_hash():
        return None
    return int(fields["traffic_bytes_per_launch"])


# VALU lane operations per 16-byte block of the default T-table launch at
# 8 MiB, table fill and per-wave setup included: rocprofv3 SQ_INSTS_VALU x 64
# / blocks (two-table layout, 512-thread workgroups, two per CU, each wave
# computing its first chunk's group constants).
VALU_PER_BLOCK_8MIB = {128: 329.0, 256: 449.0}
# VALU lane operations per block of the kernels without LDS tables: the
# bitsliced and the vector-permute kernels (rocprofv3 SQ_INSTS_VALU at 256 MiB).
VALU_PER_BLOCK_BS = {128: 678, 256: 934}
VALU_PER_BLOCK_VP = {128: 2047, 256: 2905}


def valu_roofline(args, gbs, cus, clk):
    """The T-table kernel's second ceiling at 8 MiB: VALU issue at the
    measured lane operations per block (its LDS-issue ceiling is `roofline`)."""
    if args.variant in (2, 3) or args.size != 8 * MiB:
        return {}
    v = VALU_PER_BLOCK_8MIB[args.bits]
    peak = cus * 64 * clk / v * 16 / 1e9
    return {"valu_roofline": {"bound": "valu", "achieved": round(gbs, 3), "peak": round(peak, 1), "unit": "GB/s",
                              "frac": round(gbs / peak, 4),
                              "note": f"{v} VALU lane-ops per block (rocprofv3 SQ_INSTS_VALU, fill and setup "
                                      f"included) at 64 lane-ops per clock per CU"}}


def _cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def openssl_ctr_context(size, bits, threads, seconds=3.0):
    """Labelled context, not the baseline: OpenSSL's EVP AES-CTR (AES-NI on
    the host) over 8 MiB buffers on all host threads, as the paper notes that
    AES-NI rivals a GPU on this cipher.  None if libcrypto is missing."""
    import ctypes
    import ctypes.util
    from concurrent.futures import ThreadPoolExecutor
    try:
        L = ctypes.CDLL(ctypes.util.find_library("crypto") or "libcrypto.so.3")
    except OSError:
        return None
    L.EVP_CIPHER_CTX_new.restype = ctypes.c_void_p
    L.EVP_CIPHER_CTX_free.argtypes = [ctypes.c_void_p]
    getattr(L, f"EVP_aes_{bits}_ctr").restype = ctypes.c_void_p
    L.EVP_EncryptInit_ex.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_char_p,
                                     ctypes.c_char_p]
    L.EVP_EncryptUpdate.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_int),
                                    ctypes.c_void_p, ctypes.c_int]
    key, iv = bytes(range(bits // 8)), bytes(16)
    src = ctypes.create_string_buffer(size)

    def work(_):
        ctx = L.EVP_CIPHER_CTX_new()
        dst = ctypes.create_string_buffer(size)
        outl = ctypes.c_int()
        L.EVP_EncryptInit_ex(ctx, getattr(L, f"EVP_aes_{bits}_ctr")(), None, key, iv)
        done, t0 = 0, time.perf_counter()
        while time.perf_counter() - t0 < seconds:
            L.EVP_EncryptUpdate(ctx, dst, ctypes.byref(outl), src, size)
            done += size
        L.EVP_CIPHER_CTX_free(ctx)
        return done, time.perf_counter() - t0

    with ThreadPoolExecutor(threads) as ex:
        res = list(ex.map(work, range(threads)))
    return {"gbps": round(sum(d for d, _ in res) / max(t for _, t in res) / 1e9, 2), "threads": threads,
            "kind": "OpenSSL EVP AES-CTR (AES-NI), labelled context only"}


def tune_source(A, variant, bits, size, shape=None):
    """Where a launch shape comes from: the library reads the autotuner's
    cache (AESCTR_TUNE_CACHE, else tune_cache.json beside libaesctr.so) and
    takes the entry of the same variant and key size whose size_log2 is
    floor(log2(size)), the T-table kernel's only if its grid takes the message
    in as many chunks as the size it was tuned at; without one it keeps its
    built-in rule.  Reports that
    entry, the cache's timestamp, and whether the shape in use is the entry's
    (variant 10 is the batch kernel's tiling)."""
    path = os.environ.get("AESCTR_TUNE_CACHE") or os.path.join(os.path.dirname(A._native.LIB_PATH),
                                                              "tune_cache.json")
    try:
        with open(path) as f:
            cache = json.load(f)
    except (OSError, ValueError):
        return {"source": "built-in rule (no tune cache)"}
    want = max(size, 1).bit_length() - 1
    best = None
    for e in cache.get("entries", []):
        if e.get("variant") == variant and (variant == 10 or (e.get("key_bits") == bits
                                                              and e.get("size_log2") == want)):
            best = e
            break
    if best is None:
        return {"source": "built-in rule (no matching entry)", "cache": os.path.basename(path)}
    out = {"source": "autotuner cache", "cache": os.path.basename(path), "generated": cache.get("generated"),
           "entry": best}
    if shape is not None and variant == 1:
        out["shape_matches_entry"] = (shape["blocks_per_lane"] == best["bpl"] and shape["wg_size"] == best["wg"]
                                      and shape["lds_copies"] == best["copies"]
                                      and shape["lds_tables"] == best["tables"]
                                      and shape["wave_groups"] == best.get("first", shape["wave_groups"]))
    return out


def cpu_baseline(W, size, bits, seconds):
    """The oracle, untuned, on the host cores: repeated passes over one
    benchmark buffer with all threads (median pass rate over about
    `seconds`), plus a single-thread figure on a 1 MiB slice."""
    import numpy as np
    import oracle
    key, nonce = W.sweep_key(bits)
    payload = W.sweep_payload(size, bits)
    out = np.empty_like(payload)
    threads = int(os.environ.get("OMP_NUM_THREADS") or os.cpu_count() or 1)
    oracle.ctr_mt_timed(key, nonce, 1, payload[:4096], out[:4096], threads)   # load + warm
    rates, done, t0 = [], 0, time.perf_counter()
    used = threads
    while True:
        t1 = time.perf_counter()
        used = oracle.ctr_mt_timed(key, nonce, 1, payload, out, threads)
        rates.append(size / (time.perf_counter() - t1))
        done += size
        if time.perf_counter() - t0 >= seconds:
            break
    el = time.perf_counter() - t0
    one = payload[:MiB]
    t1 = time.perf_counter()
    oracle.ctr_mt_timed(key, nonce, 1, one, out[:MiB], 1)
    single = one.size / (time.perf_counter() - t1)
    return {"value": round(_median(rates) / 1e9, 6), "unit": "GB/s", "cores": used, "kind": "oracle",
            "sample": f"{done // size} x {size // MiB} MiB AES-{bits}-CTR buffers of the benchmark "
                      f"workload through the multithreaded oracle ({el:.1f} s); median pass rate",
            "single_thread_gbps": round(single / 1e9, 6), "cpu_model": _cpu_model(),
            "host_cpus": os.cpu_count(), "openssl_context": openssl_ctr_context(size, bits, threads)}


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "one GPU only: --gpus must be 1 (the path shards by request "
                          "on the host; a multi-GPU run is not implemented)"}))
        sys.exit(2)
    import torch
    import workloads as W
    import paper_2607_02630_amd as A

    if not torch.cuda.is_available():
        print(json.dumps({"error": "no GPU visible"}))
        sys.exit(1)
    torch.cuda.set_device(0)
    props = torch.cuda.get_device_properties(0)
    cus = props.multi_processor_count
    key, nonce = W.sweep_key(args.bits)
    sched = A.aes_expand_key(key)
    cfg = A.launch_cfg(variant=args.variant) if args.variant else None

    payload, ins, outs = make_buffers(torch, W, args.size, args.bits)
    # Parity gate on the exact launch configuration being timed.
    A.aes_ctr_crypt(sched, nonce, 1, ins[0], outs[0], cfg=cfg)
    torch.cuda.synchronize()
    digest = hashlib.sha256(outs[0].cpu().numpy().tobytes()).hexdigest()
    with open(os.path.join(HERE, "tests", "golden", "ctr_digests.json")) as f:
        gold = json.load(f)["sweep"].get(f"{args.bits}/{args.size}")
    parity = None if gold is None else (digest == gold)
    if parity is False:
        print(json.dumps({"error": "GPU output differs from the oracle digest"}))
        sys.exit(3)
    log(f"parity vs oracle digest: {parity}; {len(ins)} buffer pairs")

    K = args.launches or launches_for(torch, A, sched, nonce, ins, outs, cfg)
    t = replayed_steps(torch, A, sched, nonce, ins, outs, K, args.steps, args.warmup, cfg)
    ms_per_step = t.ms / args.steps
    us_per_launch = t.ms * 1e3 / (args.steps * K)
    gbs = args.size / (us_per_launch * 1e-6) / 1e9
    log(f"steady state: {args.steps} steps of {K} launches, {ms_per_step:.2f} ms/step, "
        f"{us_per_launch:.3f} us/launch, {gbs:.1f} GB/s (wall {t.wall_ms:.1f} ms)")
    te = eager(torch, A, sched, nonce, ins, outs, 2000, cfg)
    eager_gbs = args.size * 2000 / (te.ms * 1e-3) / 1e9
    lat = single_latency_us(torch, A, sched, nonce, ins[0], outs[0], cfg=cfg)
    e2e, e2e_out = end_to_end_gbs(torch, A, sched, nonce, payload)
    pipe = {f"{c // 1024} KiB": round(end_to_end_pipelined_gbs(torch, A, sched, nonce, payload, e2e_out, chunk=c), 3)
            for c in (512 * 1024, 1 * MiB, 2 * MiB) if c < len(payload)}
    e2e_pipe = max(pipe.values()) if pipe else e2e
    e2e_zc, e2e_zc_us = end_to_end_zero_copy_gbs(torch, A, sched, nonce, payload, e2e_out)
    del e2e_out
    log(f"eager {eager_gbs:.1f} GB/s, single launch {lat:.1f} us, end-to-end {e2e:.2f} GB/s "
        f"(pipelined copies {e2e_pipe:.2f}, zero-copy {e2e_zc:.2f})")

    # Warm: the same buffer pair every launch (in + out stay in the 256 MB
    # Infinity Cache); reported beside the cold figure, never as `value`.
    tw = replayed_steps(torch, A, sched, nonce, ins[:1], outs[:1], K, 3, 1, cfg)
    warm_gbs = args.size * 3 * K / (tw.ms * 1e-3) / 1e9

    # Roofline of the dominant kernel: algorithmic bytes per launch = 2 x size
    # (payload in + out); average launch duration from the events above.
    hbm_achieved = 2 * args.size / (us_per_launch * 1e-6) / 1e9
    nr = 10 if args.bits == 128 else 14
    # Roofline of the cipher kernel.  T-table kernel: bound by LDS issue;
    # gfx950 reads 128 B/clk per CU from LDS (32 banks x 4 B), i.e. 32 random
    # 4-byte lookups per clock.  The unit of work is the method's: 16*Nr table
    # lookups per 16-byte block (160 for AES-128, 224 for AES-256), so the
    # peak is 256 CUs x 2.4 GHz x 32 / (16*Nr) blocks per second.  With
    # counter-mode caching of rounds 1-2 this kernel does 27 fewer (133 /
    # 197); the ceiling at that count is in the note.  The bitsliced kernel
    # has no lookups and is bound by VALU issue (64 lane-ops per clock per CU,
    # at its own instruction count per block).
    clk = 2.4e9
    if args.variant in (2, 3):
        valu_per_block = (VALU_PER_BLOCK_BS if args.variant == 2 else VALU_PER_BLOCK_VP)[args.bits]
        alu_peak_gbs = cus * 64 * clk / valu_per_block * 16 / 1e9
        alu_note = f"payload GB/s vs the VALU-issue ceiling of {valu_per_block} ops per block"
    else:
        lookups = 16 * nr - 27
        alu_peak_gbs = cus * clk * 32 / (16 * nr) * 16 / 1e9
        cached_peak = cus * clk * 32 / lookups * 16 / 1e9
        alu_note = (f"payload GB/s vs the LDS-issue ceiling at the method's 16*Nr = {16 * nr} table lookups "
                    f"per block; at the kernel's own {lookups} (counter-mode caching of rounds 1-2) the "
                    f"ceiling is {cached_peak:.1f} GB/s")
    result = {
        "metric": "AES-CTR GB/s at 1/8 MiB; batched GB/s + p99 latency vs per-request launch",
        "value": round(gbs, 3),
        "unit": "GB/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u8",
        "data": "synthetic: seeded uniform random bytes (PCG64), seeded key/nonce, ctr0=1",
        "config": {"workload": f"AES-{args.bits}-CTR single buffer {args.size // MiB} MiB, "
                               "kernel-only steady state, cold buffers (sweep 4 KiB-8 MiB + 256 MiB "
                               "in 'sweep')",
                   "key_bits": args.bits, "buffer_bytes": args.size, "buffers_rotated": len(ins),
                   "launches_per_step": K,
                   "timed_launch": f"each step replays a captured HIP graph of {K} launches "
                                   f"({us_per_launch:.3f} us each)",
                   "parity_vs_oracle_digest": parity,
                   "shape": A.launch_shape(args.bits, args.size, cfg),
                   "shape_source": tune_source(A, args.variant or 1, args.bits, args.size,
                                               A.launch_shape(args.bits, args.size, cfg))},
        "roofline": {"bound": "alu", "achieved": round(gbs, 3), "peak": round(alu_peak_gbs, 1),
                     "unit": "GB/s", "frac": round(gbs / alu_peak_gbs, 4),
                     "traffic": measured_traffic(args.bits, args.size, args.variant),
                     "note": alu_note},
        "hbm_roofline": {"bound": "hbm", "achieved": round(hbm_achieved, 1), "peak": HBM_PEAK_GBS,
                         "unit": "GB/s", "frac": round(hbm_achieved / HBM_PEAK_GBS, 4)},
        **valu_roofline(args, gbs, cus, clk),
        "eager_gbs": round(eager_gbs, 3),
        "warm_gbs": round(warm_gbs, 3),
        "single_launch_latency_us": round(lat, 2),
        "end_to_end_pinned_gbs": round(e2e, 3),
        "end_to_end_pinned_pipelined_gbs": round(e2e_pipe, 3),
        "end_to_end_pipelined_by_chunk": pipe,
        "end_to_end_pinned_zero_copy_gbs": round(e2e_zc, 3),
        "end_to_end_zero_copy_request_us": e2e_zc_us,
        "device": {"name": props.name, "cus": cus},
    }
    # The metric's other size: 1 MiB, same key, kernel-only steady state over
    # cold rotated buffers, after a parity check against the stored digest.
    if args.size == 8 * MiB and args.variant == 0:
        result["at_1MiB"] = one_mib_leg(torch, A, W, sched, nonce, args)

    # Calibration for HBM-traffic counters: a plain copy of the same size
    # (torch's copy kernel) moves exactly size bytes in and size bytes out.
    for _ in range(5):
        outs[1].copy_(ins[1])
    torch.cuda.synchronize()
    del ins, outs
    torch.cuda.empty_cache()

    if args.sweep:
        result["sweep"] = run_sweep(torch, A, W, args)
    if not args.no_batch:
        result["batch"] = batch_leg(torch, A, W)
    if not args.no_serve:
        result["serving"] = serve_leg(torch, A, W, args.serve_requests)
    if not args.no_hash:
        result["hash"] = hash_leg(torch, A, W, with_cpu=not args.no_cpu)
    if not args.no_aio:
        result["aio"] = aio_leg(torch)
    if not args.no_cpu:
        log("cpu baseline (oracle)")
        result["cpu_baseline"] = cpu_baseline(W, args.size, args.bits, args.cpu_seconds)
    print(json.dumps(result), flush=True)


def one_mib_leg(torch, A, W, sched, nonce, args):
    size = MiB
    payload, ins, outs = make_buffers(torch, W, size, args.bits)
    A.aes_ctr_crypt(sched, nonce, 1, ins[0], outs[0])
    torch.cuda.synchronize()
    digest = hashlib.sha256(outs[0].cpu().numpy().tobytes()).hexdigest()
    with open(os.path.join(HERE, "tests", "golden", "ctr_digests.json")) as f:
        gold = json.load(f)["sweep"][f"{args.bits}/{size}"]
    if digest != gold:
        raise SystemExit("1 MiB output differs from the oracle digest")
    K = launches_for(torch, A, sched, nonce, ins, outs)
    t = replayed_steps(torch, A, sched, nonce, ins, outs, K, args.steps, args.warmup)
    us = t.ms * 1e3 / (args.steps * K)
    shape = A.launch_shape(args.bits, size)
    out = {"gbps": round(size / (us * 1e-6) / 1e9, 3), "us_per_launch": round(us, 3), "steps": args.steps,
           "launches_per_step": K, "buffers_rotated": len(ins), "parity_vs_oracle_digest": True, "shape": shape,
           "shape_source": tune_source(A, 1, args.bits, size, shape)}
    log(f"1 MiB: {args.steps} steps of {K} launches, {us:.3f} us/launch, {out['gbps']:.1f} GB/s")
    del ins, outs
    torch.cuda.empty_cache()
    return out


def run_sweep(torch, A, W, args):
    with open(os.path.join(HERE, "tests", "golden", "ctr_digests.json")) as f:
        gold = json.load(f)["sweep"]
    out = {}
    for bits in (128, 256):
        key, nonce = W.sweep_key(bits)
        sched = A.aes_expand_key(key)
        for size in W.SWEEP_SIZES + [W.BIG_SIZE]:
            for variant in (1, 2, 3):
                cfg = A.launch_cfg(variant=variant)
                payload, ins, outs = make_buffers(torch, W, size, bits)
                # Parity gate on this exact (variant, key size, size) before it is timed.
                A.aes_ctr_crypt(sched, nonce, 1, ins[0], outs[0], cfg=cfg)
                torch.cuda.synchronize()
                digest = hashlib.sha256(outs[0].cpu().numpy().tobytes()).hexdigest()
                if digest != gold[f"{bits}/{size}"]:
                    raise SystemExit(f"sweep: variant {variant} AES-{bits} {size} B differs from the oracle digest")
                steps = max(20, min(2000, int(16e9 / size)))   # replays of >= ~10 ms, like the headline
                t, _ = steady_state(torch, A, sched, nonce, ins, outs, steps, 10, cfg, repeats=3)
                ms = t.ms / steps
                lat = single_latency_us(torch, A, sched, nonce, ins[0], outs[0], reps=20, cfg=cfg)
                row = {"kernel_gbs": round(size / (ms * 1e-3) / 1e9, 3), "us_per_launch": round(ms * 1e3, 3),
                       "single_launch_us": round(lat, 2), "parity_vs_oracle_digest": True}
                if variant == 1:
                    row["end_to_end_pinned_gbs"] = round(end_to_end_gbs(torch, A, sched, nonce, payload)[0], 3)
                name = {1: "tt", 2: "bs", 3: "vp"}[variant]
                out[f"aes{bits}/{name}/{size}"] = row
                log(f"sweep {bits} {name} {size}: {row}")
                del ins, outs
                torch.cuda.empty_cache()
    return out


def _median(xs):
    xs = sorted(xs)
    return xs[len(xs) // 2]


def batch_leg(torch, A, W, reps=5):
    """4096 requests, log-uniform 4 KiB..8 MiB, mixed AES-128/256 keys, own
    nonce and counter each: one aes_ctr_crypt_batch (upload of the
    descriptor table + one persistent kernel) vs 4096 aes_ctr_crypt
    launches (eager, graph-replayed) and vs synchronising after each."""
    import numpy as np
    import oracle
    reqs = W.batch_requests()
    offs, pos = [], 0
    for r in reqs:
        offs.append(pos)
        pos += (r.length + 255) // 256 * 256
    total = sum(r.length for r in reqs)
    log(f"batch leg: {len(reqs)} requests, {total / 2**30:.2f} GiB")
    src = W.device_payload(pos, 4242)
    dst = torch.zeros_like(src)
    t0 = time.perf_counter()
    scheds = [A.aes_expand_key(r.key) for r in reqs]
    expand_us = (time.perf_counter() - t0) / len(reqs) * 1e6
    objs = [A.Request(s, r.nonce, r.ctr0, src.data_ptr() + o, dst.data_ptr() + o, r.length)
            for s, r, o in zip(scheds, reqs, offs)]
    arr = A.make_desc_array(objs)
    st = torch.cuda.current_stream().cuda_stream
    n = len(reqs)

    def batched():
        rc = A.lib.aes_ctr_crypt_batch(arr, n, st)
        assert rc == 0, A.aes_strerror(rc)

    for _ in range(2):
        batched()
    ms = []
    for _ in range(reps):
        with Timer(torch) as t:
            batched()
        ms.append(t.ms)
    b_ms = _median(ms)
    # Parity gate: first and last block of 256 sampled requests vs the oracle.
    rng = np.random.default_rng(7)
    for i in rng.choice(n, 256, replace=False):
        r, o = reqs[i], offs[i]
        nb = (r.length + 15) // 16
        for j in (0, nb - 1):
            a, b = o + 16 * j, min(o + 16 * j + 16, o + r.length)
            ref = oracle.ctr(r.key, r.nonce, (r.ctr0 + j) & 0xFFFFFFFF, src[a:b].cpu().numpy())
            if not np.array_equal(dst[a:b].cpu().numpy(), ref):
                raise SystemExit(f"batch output differs from the oracle (request {i}, block {j})")

    args = [(ctypes_byref(s), r.nonce, r.ctr0 & 0xFFFFFFFF, src.data_ptr() + o, dst.data_ptr() + o, r.length)
            for s, r, o in zip(scheds, reqs, offs)]

    def per_request(sync=False):
        for a in args:
            A.lib.aes_ctr_crypt(*a, st)
            if sync:
                torch.cuda.synchronize()

    per_request()
    ms = []
    for _ in range(reps):
        with Timer(torch) as t:
            per_request()
        ms.append(t.ms)
    e_ms = _median(ms)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cst = torch.cuda.current_stream().cuda_stream
        for a in args:
            A.lib.aes_ctr_crypt(*a, cst)
    g.replay()
    ms = []
    for _ in range(reps):
        with Timer(torch) as t:
            g.replay()
        ms.append(t.ms)
    gr_ms = _median(ms)
    with Timer(torch) as t:
        per_request(sync=True)
    s_ms = t.ms
    out = {"requests": n, "bytes": total, "key_bits": "2048 x 128 + 2048 x 256",
           "batched_ms": round(b_ms, 3), "batched_gbps": round(total / b_ms / 1e6, 2),
           "per_request_launch_ms": round(e_ms, 3), "per_request_launch_gbps": round(total / e_ms / 1e6, 2),
           "per_request_graph_ms": round(gr_ms, 3), "per_request_graph_gbps": round(total / gr_ms / 1e6, 2),
           "sync_per_request_ms": round(s_ms, 3), "sync_per_request_gbps": round(total / s_ms / 1e6, 2),
           "speedup_vs_launches": round(e_ms / b_ms, 2), "speedup_vs_graph_launches": round(gr_ms / b_ms, 2),
           "key_expansion_us_per_key": round(expand_us, 2), "parity_sampled_vs_oracle": True,
           "tiling_source": tune_source(A, 10, 0, 0)}
    log(f"batch leg: {out}")
    del g, src, dst
    torch.cuda.empty_cache()
    return out


def ctypes_byref(x):
    import ctypes
    return ctypes.byref(x)


def hash_leg(torch, A, W, with_cpu=True, reps=5):
    """Batched SHA-256 (the second pure offload): 262,144 device-resident
    messages of 4 KiB (1 GiB) hashed by one sha256_batch call.  The timed
    call includes staging the 8 MiB descriptor table over PCIe; kernel-only
    time is in the rocprofv3 summary.  Sampled digests are checked against
    hashlib (the oracle's own pin); the oracle itself only runs as the CPU
    baseline.  Roofline: bound by integer VALU, about 1360
    instructions per 64-byte block (from the built kernel)."""
    import numpy as np
    n, size = W.HASH_MESSAGES, W.HASH_MESSAGE_BYTES
    src = W.device_payload(n * size, W.seed_for(7))
    dig = torch.zeros(n * 32, dtype=torch.uint8, device="cuda")
    base, dbase = src.data_ptr(), dig.data_ptr()
    descs = A.make_sha_desc_array((base + i * size, size, dbase + 32 * i) for i in range(n))
    for _ in range(2):
        A.sha256_batch(descs=descs, n=n)
    torch.cuda.synchronize()
    ms = []
    for _ in range(reps):
        with Timer(torch) as t:
            A.sha256_batch(descs=descs, n=n)
        ms.append(t.ms)
    call_ms = _median(ms)
    # Back to back: the host validates and stages a call while the GPU still
    # hashes the one before.
    k = 10
    with Timer(torch) as t:
        for _ in range(k):
            A.sha256_batch(descs=descs, n=n)
    b2b_ms = t.ms / k
    import hashlib
    idx = np.random.default_rng(11).choice(n, size=256, replace=False)
    host = src.view(n, size)[torch.from_numpy(idx).cuda()].cpu().numpy()
    d = dig.view(n, 32).cpu().numpy()
    ok = all(d[i].tobytes() == hashlib.sha256(host[k].tobytes()).digest() for k, i in enumerate(idx))
    if not ok:
        raise SystemExit("batched SHA-256 differs from hashlib")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    valu_per_block = 1360
    peak = cus * 64 * 2.4e9 / valu_per_block * 64 / 1e9
    gbs = n * size / (call_ms * 1e-3) / 1e9
    out = {"messages": n, "message_bytes": size, "call_ms": round(call_ms, 3), "gbps": round(gbs, 2),
           "messages_per_s": round(n / (call_ms * 1e-3)), "parity_sampled_vs_hashlib": ok,
           "back_to_back_call_ms": round(b2b_ms, 3), "back_to_back_gbps": round(n * size / (b2b_ms * 1e-3) / 1e9, 2),
           "roofline": {"bound": "alu", "achieved": round(gbs, 2), "peak": round(peak, 1), "unit": "GB/s",
                        "frac": round(gbs / peak, 4),
                        "note": f"{valu_per_block} VALU per 64-byte block; the call includes the descriptor upload"}}
    log(f"hash leg: {n} x {size} B in {call_ms:.3f} ms = {gbs:.1f} GB/s; back to back "
        f"{b2b_ms:.3f} ms per call")
    if with_cpu:
        from oracle import sha
        sample = np.frombuffer(np.random.default_rng(12).bytes(4096 * size), dtype=np.uint8).reshape(4096, size)
        threads = int(os.environ.get("OMP_NUM_THREADS") or os.cpu_count() or 1)
        sha.sha256_many(sample[:64], threads)
        t0, done, used = time.perf_counter(), 0, threads
        while time.perf_counter() - t0 < 3.0:
            _, used = sha.sha256_many(sample, threads)
            done += sample.nbytes
        el = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": round(done / el / 1e9, 4), "unit": "GB/s", "cores": used, "kind": "oracle",
                               "sample": f"4096 x 4 KiB messages through the multithreaded oracle ({el:.1f} s)"}
    del src, dig
    torch.cuda.empty_cache()
    return out


def serve_pinned(torch, A, W, g, n_req, npool=2000, budget=4 << 30):
    """The serving mix with payloads in pinned host memory: the engine's
    kernels read and write them over PCIe (host_buffers), against the
    synchronous path that copies each request in, encrypts it, copies it out
    and synchronises.  Points at 10/50/90% of the engine's saturation rate."""
    import numpy as np
    from paper_2607_02630_amd import loadgen
    which = g.choice(3, size=npool, p=W.SERVING_MIX)
    lens = np.array(W.SERVING_SIZES, dtype=np.int64)[which]
    offs = np.concatenate([[0], np.cumsum(lens)[:-1]])
    total = int(lens.sum())
    src = torch.empty(total, dtype=torch.uint8, pin_memory=True)
    src.numpy()[:] = np.frombuffer(g.bytes(total), dtype=np.uint8)
    dst = torch.zeros(total, dtype=torch.uint8, pin_memory=True)
    dev = torch.empty(max(W.SERVING_SIZES), dtype=torch.uint8, device="cuda")
    scheds = [A.aes_expand_key(g.bytes(16)) for _ in range(npool)]
    objs = [A.Request(s, g.bytes(12), int(g.integers(0, 1 << 32)), src.data_ptr() + int(o),
                      dst.data_ptr() + int(o), int(L)) for s, o, L in zip(scheds, offs, lens)]
    pool = A.make_desc_array(objs)
    st = torch.cuda.current_stream().cuda_stream
    out = {"requests_per_point": n_req, "pool_bytes": total}
    with A.Engine(budget_bytes=budget, n_streams=2, host_buffers=True) as eng:
        loadgen.run_engine(eng, pool, np.zeros(min(4000, n_req)))         # warm-up
        sat = loadgen.run_engine(eng, pool, np.zeros(n_req))
        rate = sat["achieved_rps"]
        out["saturation"] = {k: round(v, 3) for k, v in sat.items()}
        log(f"serving (pinned host): saturation {rate:.0f} req/s, {sat['gbps']:.1f} GB/s")
        points = []
        for frac in (0.1, 0.5, 0.9):
            arr = W.serving_trace(n_req, frac * rate)[0]
            e = loadgen.run_engine(eng, pool, arr)
            s = loadgen.run_sync_host(pool, arr[:min(n_req, 5000)], dev.data_ptr(), dev.numel(), st)
            points.append({"offered_frac": frac, "offered_rps": round(frac * rate, 1),
                           "engine": {k: round(v, 3) for k, v in e.items()},
                           "sync_per_request": {k: round(v, 3) for k, v in s.items()}})
            log(f"serving pinned {frac:.0%}: engine p50 {e['p50_us']:.0f} p99 {e['p99_us']:.0f} us "
                f"{e['gbps']:.1f} GB/s; sync p99 {s['p99_us']:.0f} us {s['gbps']:.1f} GB/s")
        out["points"] = points
    # The host buffers hold every pool entry's ciphertext: decrypting them on
    # the device (same key, nonce, counter) must give the plaintext back.
    torch.cuda.synchronize()
    dct = dst.cuda()
    back = torch.empty_like(dct)
    for o in objs:
        off = o.out - dst.data_ptr()
        A.aes_ctr_crypt(o.sched, o.nonce, o.ctr0, dct.data_ptr() + off, back.data_ptr() + off, length=o.length)
    torch.cuda.synchronize()
    out["roundtrip_ok"] = bool(torch.equal(back.cpu(), src))
    if not out["roundtrip_ok"]:
        raise SystemExit("pinned-host serving outputs do not decrypt to their inputs")
    del src, dst, dct, back, dev
    return out


def tenant_key_points(torch, A, W, src, dst, lens, offs, rate, n_req, n_keys=64, slots=64):
    """The serving mix with keys that repeat: every request uses one of 64
    tenant keys (own nonce and counter).  One engine keeps the schedules in
    64 resident key slots, another carries every key inline; both replay the
    same open-loop schedules at 50% and 90% of the saturation rate."""
    import numpy as np
    from paper_2607_02630_amd import loadgen
    g = np.random.default_rng(W.seed_for(6))
    dst = torch.zeros_like(dst)         # its own outputs
    torch.cuda.synchronize()
    scheds = [A.aes_expand_key(g.bytes(16)) for _ in range(n_keys)]
    which = g.integers(0, n_keys, size=len(lens))
    objs = [A.Request(scheds[int(k)], g.bytes(12), int(g.integers(0, 1 << 32)), src.data_ptr() + int(o),
                      dst.data_ptr() + int(o), int(L)) for k, o, L in zip(which, offs, lens)]
    pool = A.make_desc_array(objs)
    out = {"tenant_keys": n_keys, "key_slots": slots, "requests_per_point": n_req}
    for name, ks in (("resident", slots), ("inline", 0)):
        with A.Engine(n_streams=2, key_slots=ks) as eng:
            loadgen.run_engine(eng, pool, np.zeros(min(20000, n_req)))
            pts = []
            for frac in (0.5, 0.9):
                arr = W.serving_trace(n_req, frac * rate)[0]
                e = loadgen.run_engine(eng, pool, arr)
                st = eng.stats()
                hits, misses = st["key_hits"], st["key_misses"]
                pts.append({"offered_frac": frac, "offered_rps": round(frac * rate, 1),
                            "engine": {k: round(v, 3) for k, v in e.items()},
                            "key_hits": hits, "key_misses": misses,
                            "hit_rate": round(hits / max(1, hits + misses), 4)})
                log(f"tenant keys, {name}, {frac:.0%}: p50 {e['p50_us']:.0f} p99 {e['p99_us']:.0f} us, "
                    f"key hits {hits} / {hits + misses}")
            out[name] = pts
    # Outputs of the tenant-key pool equal the single-request call.
    torch.cuda.synchronize()
    alone = torch.zeros_like(dst)
    for o in objs:
        A.aes_ctr_crypt(o.sched, o.nonce, o.ctr0, o.x, alone.data_ptr() + (o.out - dst.data_ptr()),
                        length=o.length)
    torch.cuda.synchronize()
    out["same_alone_and_in_the_mix"] = bool(torch.equal(alone, dst))
    if not out["same_alone_and_in_the_mix"]:
        raise SystemExit("tenant-key serving outputs differ from the single-request outputs")
    del alone, dst
    torch.cuda.empty_cache()
    return out


def aio_leg(torch, sizes=(4096, MiB, 8 * MiB), clients=50, seconds=1.0):
    """The shape of the paper's Appendix A, Table 2 on this GPU: one asyncio
    event loop serving 50 closed-loop clients, each request doing a little
    CPU work plus one AES-CTR offload of the block size, served
    synchronously (the offload blocks the loop) and rerouted (submit, await
    the engine's completion, resume), in requests per second."""
    import asyncio
    from paper_2607_02630_amd import aio
    rows = []
    for size in sizes:
        sync = asyncio.run(aio._serve("sync", size, clients, seconds, torch))
        asy = asyncio.run(aio._serve("async", size, clients, seconds, torch))
        rows.append({"block_bytes": size, "sync_rps": round(sync, 1), "async_rps": round(asy, 1),
                     "speedup": round(asy / sync, 2)})
        log(f"aio {size} B: sync {sync:.0f} req/s, rerouted {asy:.0f} req/s")
    torch.cuda.empty_cache()
    return {"clients": clients, "seconds_per_point": seconds, "rows": rows}


def serve_leg(torch, A, W, n_req=100_000, budget=4 << 30):
    """Open-loop Poisson arrivals at 10/50/90% of the engine's measured
    saturation rate on the serving mix (70% 64 KiB / 25% 1 MiB / 5% 8 MiB,
    per-request AES-128 key, nonce, counter), device-resident payloads and a
    4 GiB admission budget; latency from scheduled arrival to completion.
    The synchronous per-request path (launch + synchronise, one at a time)
    replays the same schedules."""
    import numpy as np
    from paper_2607_02630_amd import loadgen
    g = np.random.default_rng(W.seed_for(5))
    npool = 12000
    which = g.choice(3, size=npool, p=W.SERVING_MIX)
    lens = np.array(W.SERVING_SIZES, dtype=np.int64)[which]
    offs = np.concatenate([[0], np.cumsum(lens)[:-1]])
    total = int(lens.sum())
    log(f"serving leg: pool of {npool} requests, {total / 2**30:.2f} GiB")
    src = W.device_payload(total, 555)
    dst = torch.zeros_like(src)
    torch.cuda.synchronize()        # the engine's streams are not ordered after torch's
    scheds = [A.aes_expand_key(g.bytes(16)) for _ in range(npool)]
    objs = [A.Request(s, g.bytes(12), int(g.integers(0, 1 << 32)), src.data_ptr() + int(o),
                      dst.data_ptr() + int(o), int(L)) for s, o, L in zip(scheds, offs, lens)]
    pool = A.make_desc_array(objs)
    out = {"budget_bytes": budget, "mix": "70% 64 KiB / 25% 1 MiB / 5% 8 MiB", "requests_per_point": n_req,
           "payloads": "device-resident"}
    with A.Engine(budget_bytes=budget, n_streams=2) as eng:
        loadgen.run_engine(eng, pool, np.zeros(min(20000, n_req)))        # warm-up
        sat = loadgen.run_engine(eng, pool, np.zeros(n_req))
        out["saturation"] = {k: round(v, 3) for k, v in sat.items()}
        rate = sat["achieved_rps"]
        log(f"serving: saturation {rate:.0f} req/s, {sat['gbps']:.1f} GB/s")
        points = []
        for frac in (0.1, 0.5, 0.9):
            arr = W.serving_trace(n_req, frac * rate)[0]
            e = loadgen.run_engine(eng, pool, arr)
            s = loadgen.run_sync(pool, arr[:min(n_req, 20000)], torch.cuda.current_stream().cuda_stream)
            points.append({"offered_frac": frac, "offered_rps": round(frac * rate, 1),
                           "engine": {k: round(v, 3) for k, v in e.items()},
                           "sync_per_request": {k: round(v, 3) for k, v in s.items()}})
            log(f"serving {frac:.0%}: engine p50 {e['p50_us']:.0f} p99 {e['p99_us']:.0f} us {e['gbps']:.1f} GB/s;"
                f" sync p99 {s['p99_us']:.0f} us {s['gbps']:.1f} GB/s")
        out["points"] = points
        out["engine_stats"] = {k: (round(v, 3) if isinstance(v, float) else v) for k, v in eng.stats().items()}
        # Both paths below the synchronous path's own knee: offered loads of
        # 10/50/90% of the rate the synchronous path sustains.
        m = min(n_req, 20000)
        sync_sat = loadgen.run_sync(pool, np.zeros(m), torch.cuda.current_stream().cuda_stream)
        srate = sync_sat["achieved_rps"]
        sync_points = []
        for frac in (0.1, 0.5, 0.9):
            arr = W.serving_trace(m, frac * srate)[0]
            e = loadgen.run_engine(eng, pool, arr)
            s = loadgen.run_sync(pool, arr, torch.cuda.current_stream().cuda_stream)
            sync_points.append({"offered_frac_of_sync_saturation": frac, "offered_rps": round(frac * srate, 1),
                                "engine": {k: round(v, 3) for k, v in e.items()},
                                "sync_per_request": {k: round(v, 3) for k, v in s.items()}})
            log(f"serving at {frac:.0%} of sync saturation ({frac * srate:.0f} req/s): engine p50 "
                f"{e['p50_us']:.0f} p99 {e['p99_us']:.0f} us; sync p50 {s['p50_us']:.0f} p99 {s['p99_us']:.0f} us")
        out["sync_saturation"] = {k: round(v, 3) for k, v in sync_sat.items()}
        out["sync_points"] = sync_points
    out["tenant_keys"] = tenant_key_points(torch, A, W, src, dst, lens, offs, rate, min(n_req, 50000))
    out["pinned_host"] = serve_pinned(torch, A, W, g, min(n_req, 20000))
    # Results are the same in the mix as alone: every pool entry's output.
    torch.cuda.synchronize()
    alone = torch.zeros_like(dst)
    for o in objs:
        A.aes_ctr_crypt(o.sched, o.nonce, o.ctr0, o.x, alone.data_ptr() + (o.out - dst.data_ptr()),
                        length=o.length)
    torch.cuda.synchronize()
    out["same_alone_and_in_the_mix"] = bool(torch.equal(alone, dst))
    if not out["same_alone_and_in_the_mix"]:
        raise SystemExit("serving outputs differ from the single-request outputs")
    del src, dst, alone
    torch.cuda.empty_cache()
    return out


if __name__ == "__main__":
    main()

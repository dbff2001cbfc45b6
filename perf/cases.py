"""The work that users have this library do, as cases that can be timed.

Every case goes through the package's public entry points with the default launch shapes.  Its
``kind`` is the way of calling:

* ``eager``   a loop of ``aes_ctr_crypt`` calls, one per request, from Python;
* ``graph``   the same calls captured once in a HIP graph and replayed (a launch-bound inner loop,
              and the way the benchmark measures the kernel);
* ``batch``   ``aes_ctr_crypt_batch`` over a prebuilt descriptor array;
* ``engine``  submit to an ``Engine`` and wait for every ticket;
* ``sha``     ``sha256_batch`` over a prebuilt descriptor array.

Sizes are those of the benchmark and the tests (4 KiB to 8 MiB requests, 256 MiB buffers, 4096-request
batches, 262,144 hashed messages) and ragged ones between them; payloads, keys, nonces and counters are
random, as ciphertext and compressed payloads are.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2607_02630_amd as A

KIB, MIB = 1 << 10, 1 << 20
SERVING_SIZES, SERVING_MIX = (64 * KIB, MIB, 8 * MIB), (0.70, 0.25, 0.05)


def listed():
    return [
        # A server that encrypts small replies one call at a time: latency and launches.
        dict(name="eager_4KiB", kind="eager", dist="fixed", lo=4 * KIB, hi=4 * KIB, n=16, bits=128, ctr0=1,
             offset=0, inplace=False),
        # The same loop on ordinary records of uneven size, in place, at any address.
        dict(name="eager_ragged", kind="eager", dist="log", lo=4 * KIB, hi=MIB, n=32, bits=256, ctr0=-1,
             offset=5, inplace=True),
        # The two sizes the benchmark's metric is quoted on, launches replayed over cold buffers.
        dict(name="graph_1MiB", kind="graph", dist="fixed", lo=MIB, hi=MIB, n=256, bits=128, ctr0=1, offset=0,
             inplace=False),
        dict(name="graph_8MiB", kind="graph", dist="fixed", lo=8 * MIB, hi=8 * MIB, n=64, bits=128, ctr0=1,
             offset=0, inplace=False),
        # Files cut into segments of uneven size under AES-256, each with its own start counter.
        dict(name="graph_ragged_256", kind="graph", dist="log", lo=4 * KIB, hi=8 * MIB, n=64, bits=256, ctr0=-1,
             offset=0, inplace=False),
        # One large buffer: bulk encryption of a dataset or a model file, either key size.
        dict(name="single_256MiB", kind="eager", dist="fixed", lo=256 * MIB, hi=256 * MIB, n=1, bits=128, ctr0=1,
             offset=0, inplace=False),
        dict(name="single_odd_256", kind="eager", dist="fixed", lo=100_000_007, hi=100_000_007, n=1, bits=256,
             ctr0=-1, offset=0, inplace=True),
        # Continuous batching by the caller: 4096 requests of mixed size and key length in one call.
        dict(name="batch_4096", kind="batch", dist="log", lo=4 * KIB, hi=8 * MIB, n=4096, bits=0, ctr0=-1, offset=0,
             inplace=False),
        # A moment's queue of a busy server, at any address.
        dict(name="batch_64", kind="batch", dist="log", lo=4 * KIB, hi=MIB, n=64, bits=0, ctr0=-1, offset=3,
             inplace=False),
        # The serving engine on its mix of request sizes.
        dict(name="engine_256", kind="engine", dist="serving", lo=64 * KIB, hi=8 * MIB, n=256, bits=128, ctr0=-1,
             offset=0, inplace=False),
        # Bulk hashing: 1 GiB of 4 KiB blocks, and a few thousand records of uneven size.
        dict(name="sha_262144", kind="sha", dist="fixed", lo=4 * KIB, hi=4 * KIB, n=262144, offset=0),
        dict(name="sha_ragged", kind="sha", dist="log", lo=64, hi=64 * KIB, n=4096, offset=1),
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(("eager", "graph", "graph", "batch", "batch", "engine", "sha"))
    if kind == "sha":
        # Up to 512 MiB of messages of 64 bytes to 256 KiB.
        mean = _log(rng, 64, 256 * KIB)
        n = _log(rng, 1, min(200_000, 512 * MIB // mean))
        c = dict(kind=kind, n=n, offset=rng.choice((0, 0, rng.randrange(16))))
        if rng.random() < 0.4:
            return dict(c, dist="fixed", lo=mean, hi=mean)
        return dict(c, dist="log", lo=max(1, mean // 32), hi=mean)
    bits = rng.choice((128, 256)) if kind in ("eager", "graph") else rng.choice((0, 128, 256))
    c = dict(kind=kind, bits=bits, ctr0=rng.choice((1, -1)), offset=rng.choice((0, 0, 16, rng.randrange(16))),
             inplace=rng.random() < 0.3)
    # Up to 1 GiB in all; a single call is up to 256 MiB.
    top = _log(rng, 4 * KIB, 256 * MIB if kind == "eager" else 16 * MIB)
    if kind == "eager":
        n = rng.randint(1, 2) if top > 16 * MIB else rng.randint(8, 32)
    elif kind == "graph":
        n = min(_log(rng, 16, 512), 1024 * MIB // top)
    elif kind == "batch":
        n = min(_log(rng, 2, 6000), 1024 * MIB // top)
    else:
        n = min(_log(rng, 16, 512), 1024 * MIB // top)
    if rng.random() < 0.4:
        return dict(c, dist="fixed", lo=top, hi=top, n=max(1, n))
    return dict(c, dist="log", lo=max(1, top // 256), hi=top, n=max(1, n))


def _lengths(case, u):
    """The request lengths in ascending order: a fixed share of each size of the serving mix, or log-uniform
    over the range, the i-th in the i-th of n equal parts at the place u(), so that every seed has nearly the
    same work."""
    n = case["n"]
    if case["dist"] == "fixed":
        return [case["lo"]] * n
    if case["dist"] == "serving":
        few = [round(n * p) for p in SERVING_MIX[1:]]
        return [s for s, k in zip(SERVING_SIZES, [n - sum(few)] + few) for _ in range(k)]
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    return [min(case["hi"], max(case["lo"], int(math.exp(lo + (hi - lo) * (i + u()) / n)))) for i in range(n)]


def _payload(nbytes, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    out = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    step = 1 << 28
    for a in range(0, nbytes, step):
        out[a:a + step].random_(0, 256, generator=g)
    return out


def _place(lens, offset):
    """Byte offsets of the requests in one pool, each `offset` bytes into its own 64-byte slots, and the pool's size."""
    offs, at = [], 0
    for n in lens:
        offs.append(at + offset)
        at += (n + offset + 127) // 64 * 64
    return offs, at


def prepare(case, seed):
    order = random.Random(seed)
    lens = _lengths(case, order.random)
    order.shuffle(lens)
    offs, _ = _place(lens, case["offset"])
    # The pool's size goes by the case alone: each request at the upper end of its part of the range.
    _, total = _place([n + 1 for n in _lengths(case, lambda: 1.0)], case["offset"])
    src = _payload(total, seed)
    rng = random.Random(seed + 1)
    if case["kind"] == "sha":
        digests = torch.zeros(32 * len(lens), dtype=torch.uint8, device="cuda")
        base, dbase = src.data_ptr(), digests.data_ptr()
        descs = A.make_sha_desc_array((base + o, n, dbase + 32 * i) for i, (o, n) in enumerate(zip(offs, lens)))
        return dict(kind="sha", src=src, out=digests, descs=descs, n=len(lens))

    dst = src if case["inplace"] else torch.zeros_like(src)
    key_bits = [case["bits"] or (128, 256)[i % 2] for i in range(len(lens))]
    rng.shuffle(key_bits)
    reqs = []
    for o, n, bits in zip(offs, lens, key_bits):
        sched = A.aes_expand_key(rng.randbytes(bits // 8))
        ctr0 = rng.getrandbits(32) if case["ctr0"] < 0 else case["ctr0"]
        reqs.append(A.Request(sched, rng.randbytes(12), ctr0, src[o:o + n], dst[o:o + n]))
    s = dict(kind=case["kind"], src=src, out=dst, reqs=reqs)
    if case["kind"] == "graph":
        side = torch.cuda.Stream()
        scratch = torch.empty(lens[0], dtype=torch.uint8, device="cuda")
        with torch.cuda.stream(side):
            side.wait_stream(torch.cuda.default_stream())
            r = reqs[0]
            A.aes_ctr_crypt(r.sched, r.nonce, r.ctr0, r.x, scratch)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"], stream=side):
            for r in reqs:
                A.aes_ctr_crypt(r.sched, r.nonce, r.ctr0, r.x, r.out)
    elif case["kind"] == "batch":
        s["descs"] = A.make_desc_array(reqs)
    elif case["kind"] == "engine":
        s["descs"] = [r.desc() for r in reqs]
        s["engine"] = A.Engine(n_streams=2)
    torch.cuda.synchronize()    # the engine's streams are not ordered after torch's
    return s


def run(state):
    kind = state["kind"]
    if kind == "eager":
        for r in state["reqs"]:
            A.aes_ctr_crypt(r.sched, r.nonce, r.ctr0, r.x, r.out)
    elif kind == "graph":
        state["graph"].replay()
    elif kind == "batch":
        A.aes_ctr_crypt_batch(state["reqs"], descs=state["descs"])
    elif kind == "engine":
        eng = state["engine"]
        for t in [eng.submit_desc(d) for d in state["descs"]]:
            eng.wait(t)
    else:
        A.sha256_batch(descs=state["descs"], n=state["n"])
    return state["out"]


def work(case):
    """Payload read once and results written once; the arithmetic is integer and counted as none."""
    n, lo, hi = case["n"], case["lo"], case["hi"]
    if case["dist"] == "fixed":
        mean = lo
    elif case["dist"] == "serving":
        mean = sum(s * p for s, p in zip(SERVING_SIZES, SERVING_MIX))
    else:
        mean = (hi - lo) / math.log(hi / lo) if hi > lo else lo
    if case["kind"] == "sha":
        return {"bytes": n * (mean + 32), "flops": 0}
    return {"bytes": 2 * n * mean, "flops": 0}


def exact(case, seed):
    """Ciphertext and digests are bytes: they are equal or wrong, and no value in 64 bits stands for them."""
    return None

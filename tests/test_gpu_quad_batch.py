"""Batches of at most eight small requests (the batch kernels of ctr_quad.hip and
ctr_pair.hip) at their edges: the number of requests, empty ones at every place,
partial words, blocks and workgroups, both key sizes, start counters across the
32-bit wrap, any address, in place, and both sides of the sizes at which the next
kernel takes over; bit for bit against the CPU oracle.  The engine's resident
keys too."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu

LENGTHS = [[1], [1024], [1025], [0], [0, 17, 0], [3, 0, 0, 1023], [15, 16, 17, 31, 33, 4095, 4096, 4097],
           [100] * 8, [65536, 1, 70001], [0, 0, 0, 0, 0, 0, 0, 5]]


def build(torch, A, g, lengths, inplace):
    offs, at = [], 64
    for n in lengths:
        at += int(g.integers(0, 40))
        offs.append(at)
        at += n
    data = g.integers(0, 256, size=at + 64, dtype=np.uint8)
    x = torch.from_numpy(data.copy()).cuda()
    y = x if inplace else torch.full_like(x, 0xA5)
    want = data.copy() if inplace else np.full_like(data, 0xA5)
    reqs = []
    for i, (n, o) in enumerate(zip(lengths, offs)):
        key, nonce = g.bytes((16, 32)[(i + len(lengths)) % 2]), g.bytes(12)
        ctr0 = (0xFFFFFFFF, 0xFFFFFFF0, int(g.integers(0, 1 << 32)))[i % 3]
        reqs.append(A.Request(A.aes_expand_key(key), nonce, ctr0, x[o:o + n], y[o:o + n]))
        if n:
            want[o:o + n] = oracle.ctr(key, nonce, ctr0, data[o:o + n], threads=0)
    return reqs, y, want


def limit(torch):
    return 2 * torch.cuda.get_device_properties(0).multi_processor_count     # workgroups of 64 blocks


# More requests than the argument block takes (ctr_quad_table_kernel), up to and past its 256.
TABLES = [[5] * 9, [0] * 9 + [17], [33, 0] * 20, [0, 1024, 1025, 0] * 8, [1000] * 64, [1024] * 65, [40] * 255 + [1],
          [0] * 255 + [70_001], [40] * 257, [0] * 12]


@pytest.mark.parametrize("inplace", [False, True])
def test_table_batches_match_oracle(inplace):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(21 + inplace)
    most = 1024 * limit(torch)
    for lengths in [*TABLES, [most // 16] * 16, [most // 16] * 15 + [most // 16 + 1], [most // 128 - 7] * 128]:
        log(f"quad table: {len(lengths)} requests, {sum(lengths)} bytes, in place {inplace}")
        reqs, y, want = build(torch, A, g, lengths, inplace)
        A.aes_ctr_crypt_batch(reqs)
        torch.cuda.synchronize()
        bad = np.flatnonzero(y.cpu().numpy() != want)
        assert bad.size == 0, (lengths[:4], len(lengths), int(bad[0]))


@pytest.mark.parametrize("inplace", [False, True])
def test_small_batches_match_oracle(inplace):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(11 + inplace)
    most = 1024 * limit(torch)
    for lengths in [*LENGTHS, [most], [most - 1024, 1], [most - 1024, 1025], [most // 8] * 8, [most // 8 + 1] * 8,
                    [2 * most], [2 * most - 9, 1], [0, 2 * most - 4096, 0, 4095], [2 * most - 4096, 4097],
                    [most // 4] * 8, [most // 4 - 5] * 8]:
        log(f"quad batch: {lengths}, in place {inplace}")
        reqs, y, want = build(torch, A, g, lengths, inplace)
        A.aes_ctr_crypt_batch(reqs)
        torch.cuda.synchronize()
        bad = np.flatnonzero(y.cpu().numpy() != want)
        assert bad.size == 0, (lengths, int(bad[0]))


def test_engine_bursts_install_and_reuse_keys():
    """Bursts of more than eight small requests: tables with installs and with keys read from their slots."""
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(19)
    keys = [g.bytes((16, 32)[i % 2]) for i in range(6)]
    scheds = [A.aes_expand_key(k) for k in keys]
    with A.Engine(key_slots=4) as eng:
        for burst in range(8):
            work = []
            for _ in range(60):
                i, n = int(g.integers(0, 6)), int(g.integers(1, 3000))
                nonce, ctr0 = g.bytes(12), int(g.integers(0, 1 << 32))
                data = g.integers(0, 256, size=n, dtype=np.uint8)
                x = torch.from_numpy(data).cuda()
                work.append((i, nonce, ctr0, data, x, torch.empty_like(x)))
            torch.cuda.synchronize()
            tickets = [eng.submit(A.Request(scheds[i], nonce, ctr0, x, y)) for i, nonce, ctr0, _, x, y in work]
            for t in tickets:
                eng.wait(t)
            for j, (i, nonce, ctr0, data, _, y) in enumerate(work):
                assert np.array_equal(y.cpu().numpy(), oracle.ctr(keys[i], nonce, ctr0, data)), (burst, j)


def test_explicit_grid():
    """A grid of one workgroup takes two workgroups of quads or one of pairs; more goes to the third kernel."""
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(5)
    for lengths in ([2048], [1024, 1024], [1024, 1024, 1], [2049], [4095], [4097], [4096, 1]):
        log(f"quad batch: {lengths}, grid 1")
        reqs, y, want = build(torch, A, g, lengths, False)
        A.aes_ctr_crypt_batch(reqs, cfg=A.batch_cfg(grid=1))
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), want), lengths


def test_engine_reuses_resident_keys():
    """Launches of one request each: the first of a key installs it, later ones read it from its slot."""
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(9)
    keys = [g.bytes(16), g.bytes(32), g.bytes(16)]
    scheds = [A.aes_expand_key(k) for k in keys]
    with A.Engine(key_slots=2) as eng:
        for step in range(24):
            i = int(g.integers(0, 3))
            n = int(g.integers(1, 5000)) + (600_000 if step % 4 == 3 else 0)
            nonce, ctr0 = g.bytes(12), int(g.integers(0, 1 << 32))
            data = g.integers(0, 256, size=n, dtype=np.uint8)
            x = torch.from_numpy(data).cuda()
            y = torch.empty_like(x)
            torch.cuda.synchronize()
            eng.wait(eng.submit(A.Request(scheds[i], nonce, ctr0, x, y)))
            assert np.array_equal(y.cpu().numpy(), oracle.ctr(keys[i], nonce, ctr0, data, threads=0)), (step, i, n)

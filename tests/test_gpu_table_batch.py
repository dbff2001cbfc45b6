"""The table kernel (ctr_batch_kernel) and the small batch's kernel where other tests'
batches are small enough to run with several lanes per block: partial blocks of every
length at any address and in place, one stream's slots used again for tables that grow
and shrink, and explicit tiles, each through plain launches and through the slots'
captured graphs; bit for bit against the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu


def build(torch, A, g, lengths, inplace=False):
    offs, at = [], 32
    for i, n in enumerate(lengths):
        at += i % 16 + 1
        offs.append(at)
        at += n
    data = g.integers(0, 256, size=at + 64, dtype=np.uint8)
    x = torch.from_numpy(data.copy()).cuda()
    y = x if inplace else torch.full_like(x, 0xA5)
    want = data.copy() if inplace else np.full_like(data, 0xA5)
    reqs = []
    for i, (n, o) in enumerate(zip(lengths, offs)):
        key, nonce = g.bytes((16, 32)[i % 2]), g.bytes(12)
        ctr0 = (1, 0xFFFFFFF0, int(g.integers(0, 1 << 32)))[i % 3]
        reqs.append(A.Request(A.aes_expand_key(key), nonce, ctr0, x[o:o + n], y[o:o + n]))
        if n:
            want[o:o + n] = oracle.ctr(key, nonce, ctr0, data[o:o + n], threads=0)
    return reqs, y, want


def same(y, want, what):
    bad = np.flatnonzero(y.cpu().numpy() != want)
    assert bad.size == 0, (what, int(bad[0]))


@pytest.mark.parametrize("use_graph", [0, 1])
@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("n", [7, 40])
def test_partial_blocks_at_any_address(n, inplace, use_graph):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(n)
    lengths = [16 * int(g.integers(0, 700)) + (i + 1) % 16 for i in range(n)]
    reqs, y, want = build(torch, A, g, lengths, inplace)
    log(f"table batch: {n} requests, in place {inplace}, graph {use_graph}")
    # A grid of one workgroup is past the sizes that run with several lanes per block.
    A.aes_ctr_crypt_batch(reqs, cfg=A.batch_cfg(grid=1, use_graph=use_graph))
    torch.cuda.synchronize()
    same(y, want, lengths)


@pytest.mark.parametrize("use_graph", [0, 1])
def test_slots_are_used_again_for_tables_of_other_sizes(use_graph):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(5)
    stream = torch.cuda.Stream()
    jobs = [build(torch, A, g, [int(k) for k in g.integers(1, 6000, size=n)])
            for n in (9, 700, 40, 9, 1500, 300, 12, 900, 10, 64)]
    torch.cuda.synchronize()
    log(f"slots used again: graph {use_graph}")
    for reqs, _, _ in jobs:
        A.aes_ctr_crypt_batch(reqs, stream=stream, cfg=A.batch_cfg(grid=3, use_graph=use_graph))
    torch.cuda.synchronize()
    for i, (_, y, want) in enumerate(jobs):
        same(y, want, i)


@pytest.mark.parametrize("use_graph", [0, 1])
@pytest.mark.parametrize("bpl", [1, 2])
@pytest.mark.parametrize("tile", [1024, 4096, 65536])
def test_explicit_tiles(tile, bpl, use_graph):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(tile + bpl)
    for n, top in ((8, 9000), (30, 4000), (64, 150_000)):
        reqs, y, want = build(torch, A, g, [int(k) for k in g.integers(0, top, size=n)])
        log(f"explicit tiles: {tile} bytes, {bpl} blocks per lane, {n} requests, graph {use_graph}")
        A.aes_ctr_crypt_batch(reqs, cfg=A.batch_cfg(tile_bytes=tile, blocks_per_lane=bpl, grid=37, use_graph=use_graph))
        torch.cuda.synchronize()
        same(y, want, (n, tile, bpl))

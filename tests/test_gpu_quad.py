"""The kernel for small messages (ctr_quad.hip, four lanes per block) at its
edges: partial words and blocks, workgroup and size limits, start counters
across the 32-bit wrap, unaligned and in place, an explicit grid, and a
captured graph; bit for bit against the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu

GUARD = 64


def check(torch, A, g, bits, ctr0, length, src, dst, cfg=None):
    key, nonce = g.bytes(bits // 8), g.bytes(12)
    data = g.integers(0, 256, size=length + 2 * GUARD, dtype=np.uint8)
    x = torch.from_numpy(data).cuda()
    inplace = dst is None
    y = x if inplace else torch.full_like(x, 0xA5)
    o = src if inplace else dst
    A.aes_ctr_crypt(A.aes_expand_key(key), nonce, ctr0, x.data_ptr() + src, y.data_ptr() + o, length=length, cfg=cfg)
    torch.cuda.synchronize()
    want = data.copy() if inplace else np.full_like(data, 0xA5)
    want[o:o + length] = oracle.ctr(key, nonce, ctr0, data[src:src + length])
    bad = np.flatnonzero(y.cpu().numpy() != want)
    assert bad.size == 0, (bits, ctr0, length, src, dst, int(bad[0]) - o)


@pytest.mark.parametrize("bits", [128, 256])
@pytest.mark.parametrize("src,dst", [(0, 0), (3, 8), (1, None), (16, None), (7, 2)])
def test_quad_matches_oracle(bits, src, dst):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(bits + 10 * src)
    limit = 2048 * torch.cuda.get_device_properties(0).multi_processor_count     # bytes: 128 blocks per CU
    log(f"quad: {bits} bits, offsets {src} {dst}")
    for length in [*range(1, 36), 255, 256, 257, 271, 4096, 65537, limit - 1, limit, limit + 1]:
        ctr0 = (0xFFFFFFFF, 0xFFFFFFF8, int(g.integers(0, 1 << 32)))[length % 3]
        check(torch, A, g, bits, ctr0, length, src, dst)


@pytest.mark.parametrize("grid", [1, 3, 16])
def test_explicit_grid(grid):
    """Grids that hold the message in one chunk each and grids that loop."""
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(grid)
    cfg = A.launch_cfg(variant=A.AES_VARIANT_TTABLE, blocks_per_lane=1, wg_size=256, grid=grid, lds_copies=32,
                       lds_tables=2)
    for length in (4096 * grid - 5, 4096 * grid, 4096 * grid + 1, 4096 * grid * 3 + 9):
        log(f"quad: grid {grid}, {length} bytes")
        check(torch, A, g, 128, 77, length, 5, 9, cfg)


def test_replayed_graph():
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(3)
    key, nonce = g.bytes(16), g.bytes(12)
    sched = A.aes_expand_key(key)
    x = torch.zeros(20_001, dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)
    stream = torch.cuda.Stream()
    A.aes_ctr_crypt(sched, nonce, 5, x, y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        A.aes_ctr_crypt(sched, nonce, 5, x, y)
    for _ in range(3):
        data = g.integers(0, 256, size=x.numel(), dtype=np.uint8)
        x.copy_(torch.from_numpy(data))
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), oracle.ctr(key, nonce, 5, data))

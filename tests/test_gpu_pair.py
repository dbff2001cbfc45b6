"""The kernel with two lanes per block (ctr_pair.hip) at its edges: the sizes
between which it runs, partial half blocks and blocks, workgroup limits, start
counters across the 32-bit wrap, unaligned and in place; bit for bit against
the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu

GUARD = 64


@pytest.mark.parametrize("bits", [128, 256])
@pytest.mark.parametrize("src,dst", [(0, 0), (3, 8), (1, None), (16, None), (7, 2)])
def test_pair_matches_oracle(bits, src, dst):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(bits + 10 * src)
    per_cu = 16 * torch.cuda.get_device_properties(0).multi_processor_count     # bytes: a block per CU
    log(f"pair: {bits} bits, offsets {src} {dst}")
    first, last = 128 * per_cu, 256 * per_cu
    for length in [*range(first + 1, first + 18), first + 4096, 200 * per_cu + 4103, last - 17, last - 8, last - 7, last,
                   last + 1]:
        ctr0 = (0xFFFFFFFF, 0xFFFF8000, int(g.integers(0, 1 << 32)))[length % 3]
        key, nonce = g.bytes(bits // 8), g.bytes(12)
        data = g.integers(0, 256, size=length + 2 * GUARD, dtype=np.uint8)
        x = torch.from_numpy(data).cuda()
        y = x if dst is None else torch.full_like(x, 0xA5)
        o = src if dst is None else dst
        A.aes_ctr_crypt(A.aes_expand_key(key), nonce, ctr0, x.data_ptr() + src, y.data_ptr() + o, length=length)
        torch.cuda.synchronize()
        want = data.copy() if dst is None else np.full_like(data, 0xA5)
        want[o:o + length] = oracle.ctr(key, nonce, ctr0, data[src:src + length], threads=0)
        bad = np.flatnonzero(y.cpu().numpy() != want)
        assert bad.size == 0, (ctr0, length, int(bad[0]) - o)

"""The hash kernel for few messages (three waves per 64 messages) at its edges.

The library takes it up to 128 messages per CU.  Counts around one workgroup's
64 messages and on both sides of that limit, with lengths on both sides of
every padding boundary, and a workgroup whose messages end at very different
blocks; every digest against the SHA-256 oracle.
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import sha
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 3, 4, 55, 56, 57, 63, 64, 65, 119, 120, 127, 128, 129, 191, 192, 1000, 4096, 9999]


@pytest.mark.parametrize("n,align", [(1, 0), (2, 1), (63, 0), (64, 3), (65, 0), (193, 5), ("limit", 0), ("past", 2)])
def test_counts_and_lengths(n, align):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    limit = 128 * torch.cuda.get_device_properties(0).multi_processor_count
    short = n in ("limit", "past")
    n = {"limit": limit, "past": limit + 1}.get(n, n)
    g = np.random.default_rng(n + align)
    lens = [int(g.choice(EDGES[:12] if short else EDGES)) for _ in range(n)]
    offs, at = [], 0
    for k in lens:
        at = (at + 15) // 16 * 16 + align
        offs.append(at)
        at += k
    buf = g.integers(0, 256, size=at + 1, dtype=np.uint8)
    dev = torch.from_numpy(buf).cuda()
    dig = torch.zeros(32 * n + align, dtype=torch.uint8, device="cuda")
    log(f"sha256 split: {n} messages, align {align}")
    A.sha256_batch([(dev.data_ptr() + o, k, dig.data_ptr() + align + 32 * i) for i, (o, k) in enumerate(zip(offs, lens))])
    torch.cuda.synchronize()
    h = dig.cpu().numpy()
    for i, (o, k) in enumerate(zip(offs, lens)):
        assert h[align + 32 * i:align + 32 * i + 32].tobytes() == sha.sha256(buf[o:o + k].tobytes()), (i, k)

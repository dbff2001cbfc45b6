"""The kernel for large messages (ctr_bulk.hip) at its edges: the smallest
message it takes, ragged ends, start counters at every place in a 256-counter
group and across the 32-bit wrap, unaligned and in place; bit for bit against
the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu

GUARD = 64


def shape(A, grid):
    return A.launch_cfg(variant=A.AES_VARIANT_TTABLE, blocks_per_lane=2, wg_size=1024, grid=grid, lds_copies=32,
                        lds_tables=4)


@pytest.mark.parametrize("bits", [128, 256])
@pytest.mark.parametrize("ctr0", [0, 1, 64, 200, 255, 0xFFFFFFFF, 0xFFFFFF80, 0xFFFF0003])
def test_bulk_matches_oracle(bits, ctr0):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(bits + ctr0 % 1000)
    key, nonce = g.bytes(bits // 8), g.bytes(12)
    # A grid of 2 workgroups takes 2 x 16 waves x 4 KiB and more; of 1, its 64-tile windows too.
    for grid, length, offset in [(2, 131072, 0), (2, 131072 + 4096 + 7, 5), (2, 299_993, 16), (1, 65536 + 15, 3),
                                 (1, 600_001, 0), (3, 196608 + 16 * 255 + 1, 8)]:
        buf = g.integers(0, 256, size=length + 2 * GUARD, dtype=np.uint8)
        dev = torch.from_numpy(buf).cuda()
        p = dev.data_ptr() + offset
        log(f"bulk: {bits} bits, ctr0 {ctr0:#x}, grid {grid}, {length} bytes at {offset}")
        A.aes_ctr_crypt(A.aes_expand_key(key), nonce, ctr0, p, p, length=length, cfg=shape(A, grid))
        torch.cuda.synchronize()
        want = buf.copy()
        want[offset:offset + length] = oracle.ctr(key, nonce, ctr0, buf[offset:offset + length])
        bad = np.flatnonzero(dev.cpu().numpy() != want)
        assert bad.size == 0, (grid, length, int(bad[0]) - offset)


def test_default_shape_of_large_messages():
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for n in (65536 * cus + 65537, 131072 * cus + 16, 524288 * cus + 5):
        s = A.launch_shape(256, n)
        assert (s["wg_size"], s["blocks_per_lane"], s["lds_tables"], s["grid"]) == (1024, 2, 4, cus), (n, s)

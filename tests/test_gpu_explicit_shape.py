"""Calls that name a part of the launch shape, or nothing: output against the CPU
oracle, at sizes near those where the default call changes its kernel."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [128, 256])
@pytest.mark.parametrize("per_cu,kw", [(4100, dict(blocks_per_lane=2, wave_groups=2)),
                                       (4100, dict(blocks_per_lane=1, wave_groups=1, grid=64)),
                                       (8300, dict(wg_size=256)), (8300, dict(lds_copies=64)), (300, dict(grid=1000)),
                                       (6128, dict()), (5400, dict())])
def test_a_part_of_the_shape(bits, per_cu, kw):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g = np.random.default_rng(per_cu + bits)
    n = 16 * per_cu * cus + 7
    key, nonce, ctr0 = g.bytes(bits // 8), g.bytes(12), int(g.integers(0, 1 << 32))
    data = np.frombuffer(g.bytes(n), dtype=np.uint8)
    log(f"explicit shape: {bits} bits, {n} bytes, {kw}")
    y = A.aes_ctr_crypt(A.aes_expand_key(key), nonce, ctr0, torch.from_numpy(data.copy()).cuda(), cfg=A.launch_cfg(**kw))
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), oracle.ctr(key, nonce, ctr0, data, threads=0))

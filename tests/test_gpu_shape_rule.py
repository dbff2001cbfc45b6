"""Default launch shapes of message sizes between the tuned ones, and their
output against the CPU oracle: a tuned entry stands only for messages its grid
takes in as many chunks as the size it was timed at."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu

# blocks per CU, (threads, blocks per lane, workgroups per CU at most, tables, first-chunk mode)
RULE = [(256, (256, 1, 1, 2, 2)), (257, (512, 1, 1, 2, 2)), (512, (512, 1, 1, 2, 2)), (513, (512, 2, 1, 2, 2)),
        (1025, (512, 1, 2, 2, 2)), (1537, (512, 2, 2, 2, 1)), (2049, (512, 1, 2, 2, 2)), (2561, (512, 2, 2, 2, 1)),
        (3073, (512, 2, 4, 2, 1)), (4097, (1024, 2, 1, 4, 0))]


@pytest.mark.parametrize("bits", [128, 256])
@pytest.mark.parametrize("per_cu,want", RULE)
def test_shape_and_output_between_tuned_sizes(bits, per_cu, want):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 16 * (per_cu - 1) * cus + 16 * 3 + 11     # the first CU's share is one block more
    s = A.launch_shape(bits, n)
    wg, bpl, most, tables, mode = want
    log(f"{bits} bits, {per_cu} blocks per CU: {s}")
    assert (s["wg_size"], s["blocks_per_lane"], s["lds_tables"], s["wave_groups"]) == (wg, bpl, tables, mode), s
    assert s["grid"] <= most * cus
    g = np.random.default_rng(per_cu + bits)
    key, nonce, ctr0 = g.bytes(bits // 8), g.bytes(12), int(g.integers(0, 1 << 32))
    data = np.frombuffer(g.bytes(n), dtype=np.uint8)
    y = A.aes_ctr_crypt(A.aes_expand_key(key), nonce, ctr0, torch.from_numpy(data.copy()).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), oracle.ctr(key, nonce, ctr0, data, threads=0))

"""Small batches whose tiles just fill all waves (ctr_batch_small_kernel with tiles cut
from the requests' starts, run_tile without the shift): steps over two counter
groups, windows of 64 groups, partial blocks, any address, in place, the counter's
wrap; bit for bit against the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu

# With one workgroup the kernel has 8 waves.  (requests, tiles each, tile bytes)
CASES = [(1, 8, 1024), (1, 8, 2048), (1, 16, 2048), (2, 4, 4096), (3, 8, 2048), (8, 1, 3072), (4, 2, 524288), (8, 1, 262144 + 1024),
         (8, 2, 300 * 1024)]


@pytest.mark.parametrize("bpl", [1, 2])
@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("n,tiles,tile", CASES)
def test_tiles_from_the_requests_starts(n, tiles, tile, bpl, inplace):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(n * tiles + tile + bpl)
    length = tiles * tile
    for cut in (0, 1, 15):
        offs = [i * (length + 256) + 64 + int(g.integers(0, 16)) for i in range(n)]
        data = g.integers(0, 256, size=n * (length + 256) + 128, dtype=np.uint8)
        x = torch.from_numpy(data.copy()).cuda()
        y = x if inplace else torch.full_like(x, 0xA5)
        want = data.copy() if inplace else np.full_like(data, 0xA5)
        reqs = []
        for i, o in enumerate(offs):
            key, nonce = g.bytes((16, 32)[i % 2]), g.bytes(12)
            ctr0 = (1, 0xFFFFFFC1, 255, int(g.integers(0, 1 << 26)) * 64 + 63, 0xFFFFFE01)[(i + cut) % 5]
            reqs.append(A.Request(A.aes_expand_key(key), nonce, ctr0, x[o:o + length - cut], y[o:o + length - cut]))
            want[o:o + length - cut] = oracle.ctr(key, nonce, ctr0, data[o:o + length - cut], threads=0)
        log(f"small tiles: {n} requests of {length - cut} bytes, tile {tile}, bpl {bpl}, in place {inplace}")
        A.aes_ctr_crypt_batch(reqs, cfg=A.batch_cfg(tile_bytes=tile, blocks_per_lane=bpl, grid=1))
        torch.cuda.synchronize()
        bad = np.flatnonzero(y.cpu().numpy() != want)
        assert bad.size == 0, (n, length, cut, int(bad[0]))

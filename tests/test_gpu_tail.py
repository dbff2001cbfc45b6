"""Messages that end in a partial block, at the edges of the T-table kernel's
chunks, and batch requests that do, at any address; bit for bit against the
CPU oracle.

A workgroup takes chunks of wg * blocks-per-lane blocks; the partial block is
the first or the last block of a chunk, of a wave's 64, alone in a chunk, or
the whole message, in the first chunk of a launch or a later one.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu

GUARD = 64


def run(length, bits, cfg, offset, seed):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(seed)
    key, nonce, ctr0 = g.bytes(bits // 8), g.bytes(12), int(g.integers(0, 1 << 32))
    buf = g.integers(0, 256, size=length + 2 * GUARD, dtype=np.uint8)
    dev = torch.from_numpy(buf).cuda()
    p = dev.data_ptr() + offset
    A.aes_ctr_crypt(A.aes_expand_key(key), nonce, ctr0, p, p, length=length, cfg=cfg)
    torch.cuda.synchronize()
    want = buf.copy()
    want[offset:offset + length] = oracle.ctr(key, nonce, ctr0, buf[offset:offset + length])
    got = dev.cpu().numpy()
    bad = np.flatnonzero(got != want)
    assert bad.size == 0, (length, int(bad[0]) - offset)


@pytest.mark.parametrize("bits", [128, 256])
@pytest.mark.parametrize("wg,bpl,mode", [(256, 1, 2), (512, 1, 3), (512, 2, 2), (512, 2, 1), (1024, 2, 3), (512, 4, 3)])
def test_partial_block_at_chunk_edges(bits, wg, bpl, mode):
    import paper_2607_02630_amd as A
    cfg = A.launch_cfg(variant=A.AES_VARIANT_TTABLE, blocks_per_lane=bpl, wg_size=wg, grid=2, lds_copies=32,
                       lds_tables=2, wave_groups=mode)
    chunk = wg * bpl
    log(f"partial block: {bits} bits, wg {wg}, bpl {bpl}, mode {mode}")
    for blocks, tail in [(0, 1), (0, 15), (1, 7), (63, 4), (64, 8), (chunk - 1, 3), (chunk, 12), (2 * chunk, 5),
                         (2 * chunk + 64 * bpl, 2), (3 * chunk - 1, 11), (4 * chunk, 14), (5 * chunk + 77, 13)]:
        run(16 * blocks + tail, bits, cfg, offset=(blocks + tail) % 16, seed=blocks + tail)


@pytest.mark.parametrize("n", [3, 40])
def test_batch_of_odd_requests_at_any_address(n):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(n)
    lens = [int(g.integers(1, 9000)) if i % 4 else i + 1 for i in range(n)]
    offs = np.cumsum([0] + [(k + GUARD) // 64 * 64 + 64 for k in lens]) + np.arange(n + 1) % 16
    src = g.integers(0, 256, size=int(offs[-1]) + GUARD, dtype=np.uint8)
    keys = [g.bytes(16 if i % 2 else 32) for i in range(n)]
    nonces, ctrs = [g.bytes(12) for _ in range(n)], [int(g.integers(0, 1 << 32)) for _ in range(n)]
    x = torch.from_numpy(src).cuda()
    y = torch.zeros_like(x)
    log(f"odd batch of {n}")
    A.aes_ctr_crypt_batch([A.Request(A.aes_expand_key(keys[i]), nonces[i], ctrs[i], x[int(offs[i]):int(offs[i]) + lens[i]],
                                     y[int(offs[i]) + 3:int(offs[i]) + 3 + lens[i]]) for i in range(n)])
    torch.cuda.synchronize()
    want = np.zeros_like(src)
    for i in range(n):
        o = int(offs[i])
        want[o + 3:o + 3 + lens[i]] = oracle.ctr(keys[i], nonces[i], ctrs[i], src[o:o + lens[i]])
    assert np.array_equal(y.cpu().numpy(), want)

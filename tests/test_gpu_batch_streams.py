"""Table batches from several threads on hipStreamPerThread, whose one handle is
another queue in each thread, and on streams that come and go; bit for bit against
the CPU oracle."""
from __future__ import annotations

import threading

import numpy as np
import pytest

import oracle
from gpu_util import log, torch_cuda

pytestmark = pytest.mark.gpu

PER_THREAD = 2    # hipStreamPerThread


def make(torch, A, g, lengths):
    reqs, want, outs = [], [], []
    for i, n in enumerate(lengths):
        key, nonce, ctr0 = g.bytes((16, 32)[i % 2]), g.bytes(12), int(g.integers(0, 1 << 32))
        data = g.integers(0, 256, size=n, dtype=np.uint8)
        x = torch.from_numpy(data).cuda()
        y = torch.zeros_like(x)
        reqs.append(A.Request(A.aes_expand_key(key), nonce, ctr0, x, y))
        want.append(oracle.ctr(key, nonce, ctr0, data, threads=0))
        outs.append(y)
    return reqs, A.make_desc_array(reqs), outs, want


def check(outs, want, who):
    for i, (y, w) in enumerate(zip(outs, want)):
        assert np.array_equal(y.cpu().numpy(), w), (who, i)


@pytest.mark.parametrize("use_graph", [0, 1])
def test_threads_on_the_per_thread_stream(use_graph):
    torch = torch_cuda()
    import paper_2607_02630_amd as A
    g = np.random.default_rng(use_graph)
    cfg = A.batch_cfg(use_graph=use_graph)
    jobs = [[make(torch, A, g, [int(n) for n in g.integers(1, top, size=count)])
             for count, top in ((12, 2000), (40, 200_000), (30, 5000))] for _ in range(3)]
    torch.cuda.synchronize()
    errors = []

    def work(mine):
        try:
            for _ in range(6):
                for reqs, descs, _, _ in mine:
                    A.aes_ctr_crypt_batch(reqs, stream=PER_THREAD, cfg=cfg, descs=descs)
        except Exception as e:    # noqa: BLE001
            errors.append(e)

    log(f"per-thread stream, 3 threads, graph {use_graph}")
    threads = [threading.Thread(target=work, args=(j,)) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for who, mine in enumerate(jobs):
        for _, _, outs, want in mine:
            check(outs, want, who)

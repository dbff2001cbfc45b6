"""Order of a batch call's table upload against earlier work on the same table, on
the CPU: tests/cpp/batch_order_test.cpp with the library's own batch.cpp against a
model of HIP's queues (tests/cpp/fake_hip)."""
from __future__ import annotations

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2607_02630_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("batch") / "batch_order_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-I", os.path.join(HERE, "cpp", "fake_hip"), "-I", CSRC,
                    "-o", str(out), os.path.join(HERE, "cpp", "batch_order_test.cpp"),
                    *(os.path.join(CSRC, f) for f in ("batch.cpp", "host_pool.cpp", "keys.cpp", "tune.cpp")), "-ldl"],
                   check=True)
    return str(out)


@pytest.mark.parametrize("scenario", ["handles", "failures"])
def test_uploads_wait_for_every_reader_of_the_table(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "batch order ok" in r.stdout, r.stdout + r.stderr


def routes(exe, batches):
    """[(requests, bytes, ctr0, tile_bytes, blocks_per_lane, grid, use_graph)] -> [(kernel, tiles, tile_blocks,
    workgroups, blocks_per_lane)]."""
    r = subprocess.run([exe, "routes"], input="".join(" ".join(map(str, b)) + "\n" for b in batches), capture_output=True,
                       text=True, timeout=60, check=True, env=dict(os.environ, AESCTR_TUNE_CACHE=""))
    got = [line.split() for line in r.stdout.splitlines()]
    assert len(got) == len(batches), r.stdout
    return [(g[0], *map(int, g[1:])) for g in got]


@pytest.mark.parametrize("n,size,tile", [(1, 4 << 20, 0), (4, 1 << 20, 0), (8, 512 << 10, 0), (8, 1 << 20, 0), (2, 4 << 20, 0),
                                         (1, 8 << 20, 0), (8, 8 << 20, 0), (4, 1 << 20, 2048)])
def test_a_start_counter_adds_no_round_of_tiles(exe, n, size, tile):
    """Requests that fill all waves of the small batch's kernel exactly need no further tile for a
    start counter within 64 counters: 2048 waves on 256 CUs."""
    even, odd = routes(exe, [(n, size, 0, tile, 0, 0, 0), (n, size, 1, tile, 0, 0, 0)])
    assert even[0] == "small" and even[1] % 2048 == 0, even
    assert odd[0] == "small_plain" and odd[1:3] == even[1:3], odd


@pytest.mark.parametrize("n,size,tile,bpl", [(2, 1 << 20, 0, 0), (4, 300_000, 0, 0), (4, 8192, 65536, 2), (3, 3072, 4096, 1),
                                             (1, 2 << 20, 0, 0)])
def test_a_start_counter_adds_no_step_to_one_round(exe, n, size, tile, bpl):
    even, odd = routes(exe, [(n, size, 64, tile, bpl, 0, 0), (n, size, 127, tile, bpl, 0, 0)])
    assert even[0] == "small" and even[1] <= 2048, even
    assert odd[0] == "small_plain" and odd[1:] == even[1:], odd


def test_explicit_tiles_are_the_tiles_of_the_launch(exe):
    """(requests, bytes): small enough to run with several lanes per block where the tiles are left to the library."""
    for n, size, kernel in ((1, 4096, "quad"), (8, 65536, "quad"), (1, 1 << 20, "pair"), (9, 1000, "quad_table"),
                            (200, 1500, "quad_table")):
        assert routes(exe, [(n, size, 1, 0, 0, 0, 0)])[0][0] == kernel
        for tile, bpl in ((1024, 0), (65536, 0), (0, 1), (0, 2), (4096, 1)):
            got = routes(exe, [(n, size, 0, tile, bpl, 0, 0)])[0]
            assert got[0] == ("table" if n > 8 else "small"), (n, size, tile, bpl, got)
            assert got[4] == (bpl or 2), got
            if tile:
                assert got[1:3] == (n * -(-size // tile), tile // 16), (n, size, tile, got)


def test_several_lanes_per_block_stop_at_the_chips_size(exe):
    """Quads up to two workgroups of 64 blocks per CU, pairs up to one of 256, however large the grid (256 CUs)."""
    for grid in (0, 256, 257, 4096):
        for n, size, kernel in ((8, 65536, "quad"), (4, 128 * 1024 + 1, "pair"), (4, 256 * 1024, "pair"), (4, 256 * 1024 + 1, "small"),
                                (4, 1 << 20, "small"), (16, 32768, "quad_table"), (16, 32769, "table")):
            assert routes(exe, [(n, size, 0, 0, 0, grid, 0)])[0][0] == kernel, (grid, n, size)
    for n, size, kernel in ((8, 128, "quad"), (1, 2049, "pair"), (1, 4097, "small"), (9, 200, "table")):
        assert routes(exe, [(n, size, 0, 0, 0, 1 if n == 1 else 4, 0)])[0][0] == kernel, (n, size)


def test_an_empty_configuration_is_the_default_call(exe):
    """The binding's batch_cfg() names nothing, the graph included, so few small requests keep their kernel."""
    import paper_2607_02630_amd as A
    cfg = A.batch_cfg()
    fields = (cfg.tile_bytes, cfg.blocks_per_lane, cfg.grid, cfg.use_graph)
    assert fields == (0, 0, 0, 0) and cfg.wg_size == 0
    assert routes(exe, [(64, 1000, 1, *fields)])[0][0] == "quad_table"
    assert A.batch_cfg(grid=3).use_graph == 0 and A.batch_cfg(use_graph=1).use_graph == 1

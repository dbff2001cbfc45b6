"""Which kernel and shape a single-buffer call launches, on the CPU.

Builds tests/cpp/shape_test.cpp with the library's own api.cpp, tune.cpp and
keys.cpp against a HIP runtime of host memory (tests/cpp/fake_hip, 256 CUs) and
asks it for calls under the shipped tune cache and under none.
"""
from __future__ import annotations

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2607_02630_amd", "csrc")
SHIPPED = os.path.join(HERE, "..", "paper_2607_02630_amd", "tune_cache.json")
FIELDS = ("variant", "bpl", "wg", "grid", "copies", "tables", "mode", "address")
MiB = 1 << 20


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("shape") / "shape_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(HERE, "cpp", "fake_hip"), "-I", CSRC, "-o", str(out),
                    os.path.join(HERE, "cpp", "shape_test.cpp"),
                    *(os.path.join(CSRC, f) for f in ("api.cpp", "tune.cpp", "keys.cpp")), "-ldl"], check=True)
    return str(out)


def ask(exe, calls, cache=SHIPPED):
    """[(key bits, bytes, explicit fields)] -> [(status, kernel, shape)]."""
    text = "".join(f"{bits} {n} " + " ".join(str(kw.get(f, 0)) for f in FIELDS) + "\n" for bits, n, kw in calls)
    r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60, check=True,
                       env=dict(os.environ, AESCTR_TUNE_CACHE=cache))
    got = [line.split() for line in r.stdout.splitlines()]
    assert len(got) == len(calls)
    return [(int(g[0]), g[1], tuple(map(int, g[2:]))) for g in got]


# Explicit fields that name another shape than the default's change one of the T-table
# kernel's own, whatever the default call of that size runs: (bits, bytes, fields, (bpl, wg, grid, copies, tables, mode) or None if refused).
EXPLICIT = [
    (128, 25_100_288, dict(bpl=2, mode=2), (2, 512, 1024, 32, 2, 2)),
    (128, 100_000_007, dict(bpl=1, grid=64, mode=1), (1, 512, 64, 32, 2, 1)),
    (128, 64 * MiB, dict(mode=2), None),
    (128, 16 * MiB + 100, dict(wg=512, copies=32, tables=2, mode=2), None),
    (256, 64 * MiB, dict(wg=256), (4, 256, 1024, 32, 2, 0)),
    (128, 256 * MiB, dict(wg=256), (4, 256, 1024, 32, 2, 0)),
    (256, 256 * MiB, dict(wg=512, mode=2), (1, 512, 1024, 32, 2, 2)),
    (256, 40 * MiB, dict(grid=1024), (4, 512, 1024, 32, 2, 0)),
    (128, 4_594_304, dict(grid=1024), (2, 512, 281, 32, 2, 2)),
    (128, 7_000_000, dict(copies=64), (2, 512, 256, 64, 2, 2)),
    (128, 9_000_000, dict(bpl=4), (4, 512, 275, 32, 2, 0)),
]


def test_explicit_fields_change_the_ttable_kernels_shape(exe):
    got = ask(exe, [c[:3] for c in EXPLICIT])
    for (bits, n, kw, want), (rc, kernel, shape) in zip(EXPLICIT, got):
        if want is None:
            assert rc == -1, (bits, n, kw, rc, kernel, shape)
        else:
            assert (rc, kernel, shape) == (0, "ttable", want), (bits, n, kw, rc, kernel, shape)


def test_every_mode_of_the_ttable_kernel_is_taken_at_every_size(exe, tmp_path):
    """Blocks per lane and first-chunk mode alone: what the T-table kernel's own shape
    is built for at one size of a range is taken at all of it."""
    sizes = [16 * MiB, 16 * MiB + 100, 24 * MiB - 65536, 24 * MiB, 24 * MiB + 16, 32 * MiB, 40 * MiB, 100_000_007]
    for cache in (SHIPPED, str(tmp_path / "none.json")):
        for bits in (128, 256):
            for kw in (dict(bpl=1, mode=2), dict(bpl=2, mode=1), dict(bpl=2, mode=2), dict(copies=64, bpl=2, mode=2)):
                for n, got in zip(sizes, ask(exe, [(bits, n, kw) for n in sizes], cache)):
                    assert got[:2] == (0, "ttable"), (bits, n, kw, got)


def test_fields_that_name_the_default_change_nothing(exe):
    for bits in (128, 256):
        for n in (3_000_000, 9_000_000, 20_000_003, 64 * MiB, 256 * MiB):
            default = ask(exe, [(bits, n, {})])[0]
            bpl, wg, grid, copies, tables, mode = default[2]
            for kw in (dict(bpl=bpl), dict(wg=wg, tables=tables), dict(copies=copies), dict(mode=mode or 3)):
                assert ask(exe, [(bits, n, kw)])[0] == default, (bits, n, kw)


def test_several_lanes_per_block_only_for_callers_who_name_no_shape(exe):
    """Those kernels launch workgroups of their own, more than an explicit grid holds."""
    for bits in (128, 256):
        for n, kernel in ((1, "quad"), (65536, "quad"), (512 * 1024, "quad"), (512 * 1024 + 1, "pair"), (MiB, "pair"),
                          (MiB + 1, "ttable")):
            assert ask(exe, [(bits, n, {})])[0][:2] == (0, kernel)
            assert ask(exe, [(bits, n, dict(variant=1))])[0][:2] == (0, kernel)
            named = dict(variant=1, bpl=1, wg=256, copies=32, tables=2, mode=2)
            for kw in (dict(grid=256), dict(wg=256), dict(mode=2), dict(tables=2), named, dict(named, grid=1000)):
                rc, got, shape = ask(exe, [(bits, n, kw)])[0]
                assert (rc, got) == (0, "ttable"), (bits, n, kw, got)
                assert shape[2] <= kw.get("grid", 256 + 1), (bits, n, kw, shape)


# Where the default changes between steps of a chunk per CU ("ttable", 512 threads of 4 blocks) and shared tiles ("bulk"),
# by how full the last step is: MiB on 256 CUs, for both key sizes.
STEPS = [(16, "ttable", "ttable"), (16.125, "bulk", "bulk"), (21, "bulk", "bulk"), (21.5, "bulk", "ttable"),
         (21.875, "bulk", "ttable"), (22.125, "ttable", "ttable"), (23.9375, "ttable", "ttable"), (24, "ttable", "ttable"),
         (24.125, "bulk", "bulk"), (31.5, "bulk", "bulk"), (32, "ttable", "ttable"), (32.125, "bulk", "bulk"),
         (40, "bulk", "bulk")]


def test_nearly_full_steps_keep_their_shape(exe):
    for i, bits in enumerate((128, 256)):
        for m, *kernels in STEPS:
            rc, kernel, shape = ask(exe, [(bits, int(m * MiB), {})])[0]
            assert (rc, kernel) == (0, kernels[i]), (bits, m, kernel, shape)
            assert shape[:2] == ((4, 512) if kernel == "ttable" else (2, 1024)), (bits, m, shape)


def test_two_workgroups_per_cu_below_16_mib(exe):
    """Two chunks of 512 threads x 2 blocks are resident; more workgroups in the grid fill their tables for one more."""
    for bits in (128, 256):
        for n in (11_700_000, 12 * MiB + 16, 13_700_000, 15_900_000):
            assert ask(exe, [(bits, n, {})])[0] == (0, "ttable", (2, 512, 512, 32, 2, 1)), (bits, n)


def test_steps_only_where_their_partial_blocks_and_addresses_cost_less(exe):
    """At an odd address shared tiles take less; a partial block matters to AES-128 alone."""
    for bits in (128, 256):
        assert ask(exe, [(bits, 23 * MiB, dict(address=3))])[0][1] == "bulk"
    assert ask(exe, [(128, 23 * MiB + 5, {})])[0][1] == "bulk"
    assert ask(exe, [(256, 23 * MiB + 5, {})])[0][1] == "ttable"

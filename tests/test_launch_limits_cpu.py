"""Launches of batches larger than any test can hold, recorded by a stand-in for the HIP runtime
(launch_probe.c; no GPU): every grid stays within what a launch may have."""
import os
import subprocess
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    import paper_2312_05800_amd as P
    from paper_2312_05800_amd import build
    P.lib()  # raises if the library is missing
    exe = str(tmp_path_factory.mktemp("probe") / "launch_probe")
    subprocess.check_call(["gcc", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-o", exe,
                           os.path.join(ROOT, "tests", "launch_probe.c"), "-ldl"])

    def run(call, sizes, reactions=20, lds=65536):
        """[(N, status, [(kernel, grid, block)])] of the call at every size."""
        out = subprocess.check_output([exe, build.LIB, str(lds), str(reactions), call] +
                                      [str(n) for n in sizes], text=True)
        res, launches = [], []
        for line in out.splitlines():
            w = line.split()
            if w[0] == "call":
                res.append((int(w[1]), int(w[2]), launches))
                launches = []
            else:
                launches.append((w[0], tuple(map(int, w[1:4])), tuple(map(int, w[4:7]))))
        assert [r[0] for r in res] == list(sizes)
        return res
    return run


# around 2^29 and 2^32 cells, where 8 threads or 1 thread a cell reach the limit of 2^32 - 1 in x
SIZES = [1, 64, 8191, 8192, 8193, 1 << 20, (1 << 29) - 65, (1 << 29) - 64, (1 << 29) - 63, 1 << 29,
         (1 << 30) - 1, 1 << 30, (1 << 32) - 256, (1 << 32) - 255, 1 << 32, 1 << 40]


@pytest.mark.parametrize("call", ["rates", "step", "sample"])
def test_grids_within_a_launch(probe, call):
    for n, status, launches in probe(call, SIZES):
        assert status == 0 and launches
        for name, grid, block in launches:
            assert grid[0] * block[0] < 1 << 32, (n, name, grid, block)
            assert grid[1] * block[1] < 1 << 32 and grid[2] * block[2] < 1 << 32


# 4 cells a wave, each with 16 bytes a reaction: 1024 reactions fill 64 KB, 2560 160 KB
@pytest.mark.parametrize("call", ["rates", "step"])
@pytest.mark.parametrize("lds,most", [(65536, 1024 - 32), (163840, 2560 - 32)])
def test_too_many_reactions_refused_at_every_size(probe, call, lds, most):
    sizes = [1, 8191, 8192, 1 << 20]
    assert all(st == 0 for _, st, _ in probe(call, sizes, reactions=most, lds=lds))
    for n, st, launches in probe(call, sizes, reactions=most + 33, lds=lds):
        assert st == 6 and not launches, (n, st, launches)  # CHEM_EUNSUPPORTED


def test_step_grid_can_be_resident(probe):
    """The persistent grid: what the registers allow (two waves on each of a CU's four SIMDs), however
    little LDS a mechanism needs."""
    (_, status, launches), = probe("step", [1 << 20])
    grid = [g for name, g, _ in launches if "k_step" in name]
    assert status == 0 and grid == [(256 * 8, 1, 1)]


def test_large_mechanisms_are_made_quickly(probe):
    """The order of the reactions is a search over passes; the most reactions a lane group's LDS holds
    (and as many as the descriptor may have, refused at their first use) take no minutes."""
    t0 = time.monotonic()
    probe("rates", [64], reactions=2528, lds=163840)
    probe("rates", [64], reactions=65535)
    assert time.monotonic() - t0 < 5.0

"""Launches of batches larger than any test can hold, recorded by a stand-in for the HIP runtime
(launch_probe.c; no GPU): every grid stays within what a launch may have."""
import os
import subprocess

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

"""The training tuner weighs each product with what the step then runs beside it, and both tuners'
stored results end with the kernels they were measured on.  Kernel times are set by a stand-in for
the HIP runtime (launch_probe.c; no GPU)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BATCH = 2048


@pytest.fixture(scope="module")
def tuned(tmp_path_factory):
    import paper_2312_05800_amd as P
    from paper_2312_05800_amd import build
    P.lib()  # raises if the library is missing
    tmp = tmp_path_factory.mktemp("tune")
    exe = str(tmp / "launch_probe")
    subprocess.check_call(["gcc", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-o", exe,
                           os.path.join(ROOT, "tests", "launch_probe.c"), "-ldl"])

    def call(what, cache, costs):
        env = dict(os.environ, CHEM_AUTOTUNE_CACHE=cache,
                   LAUNCH_COSTS=",".join(f"{k}={v}" for k, v in costs.items()))
        out = subprocess.check_output([exe, build.LIB, "65536", "1", what, str(BATCH)], text=True,
                                      env=env).splitlines()
        assert out[-1] == f"call {BATCH} 0", out[-1]
        return out[:-1]

    def run(**costs):
        """(tiles of the eleven products, splits of the four weight gradients, kernels launched)."""
        cache = str(tmp / ("cache" + "_".join(f"{k}{v}" for k, v in costs.items())))
        out = call("autotune_train", cache, costs)
        v = open(cache).read().split(" = ")[1].split()
        return [int(x) for x in v[0:22:2]], [int(x) for x in v[22:26]], out
    run.call, run.tmp = call, tmp
    return run


def test_data_gradients_are_charged_their_column_sums(tuned):
    """The generic tilings leave the bias gradients to a pass of their own."""
    tiles, _, _ = tuned(k_gemmI=1.0, k_gemm_dma16=1.5, k_colsum_part=2.0)
    assert tiles[8:] == [0, 0, 0]
    tiles, _, _ = tuned(k_gemmI=1.0, k_gemm_dma16=4.0, k_colsum_part=2.0)
    assert all(t > 0 for t in tiles[8:])


def test_ranges_are_added_where_the_step_adds_them(tuned):
    """k_finish adds the ranges of a split weight gradient."""
    _, splits, out = tuned(k_gemmI=1.0, k_gemm_dma16=1.0)
    assert not any("k_sum_splits" in line for line in out)
    assert any("k_finish" in line for line in out)


@pytest.mark.parametrize("what,kernel,costs", [("autotune_train", "k_gemm", dict(k_gemm=1.0)),
                                               ("autotune", "k_step", dict(k_step=1.0))])
def test_stored_results_name_their_kernels(tuned, what, kernel, costs):
    """A result is taken from the file without timing, one stored without the kernels' version is not."""
    cache = str(tuned.tmp / what)
    assert any(kernel in line for line in tuned.call(what, cache, costs))
    line = open(cache).read()
    assert not any(kernel in x for x in tuned.call(what, cache, costs))
    open(cache, "w").write(re.sub(r" v\d+ ", " ", line))
    assert any(kernel in x for x in tuned.call(what, cache, costs))
    assert line in open(cache).read()

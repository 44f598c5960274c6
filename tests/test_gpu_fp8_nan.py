"""A NaN among the inputs of the FP8 variant reaches the outputs of its own cell and no other's."""
import numpy as np
import pytest

import chemgen
from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu


# each side of the sizes where the first (6400) and the second layer's tiles change
@pytest.mark.parametrize("n", [1, 65, 2003, 6400, 6401, 30011])
def test_fp8_keeps_nan(n):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[fp8 nan] n={n}", flush=True)
    mech = chemgen.make_mechanism("ch4")
    K = mech.K
    T, p, Y = (to_dev(x, dev) for x in chemgen.make_states(mech, "ch4", N=max(n, 4096), seed=909))
    m = P.AnnModel(K + 2, K, (1600, 800, 400), seed=5)
    m.fit_norm(T, p, Y, (Y * 1.01).contiguous(), lam=0.1, dt_model=1e-5)
    m.quantize_fp8(T[:4096].contiguous(), p[:4096].contiguous(), Y[:, :4096].contiguous())
    t, q, y = T[:n].clone(), p[:n].clone(), Y[:, :n].contiguous()
    good = m.forward(t, q, y, K).cpu().numpy()
    bad = sorted({0, n // 2, n - 1})
    t[bad] = float("nan")
    u = m.forward(t, q, y, K).cpu().numpy()
    assert np.isfinite(good).all()
    assert np.isnan(u[bad]).all()
    rest = np.setdiff1d(np.arange(n), bad)
    np.testing.assert_array_equal(u[rest], good[rest])


@pytest.mark.parametrize("N", [1 << 17, (1 << 17) + 77])
def test_fp8_nan_does_not_outlive_its_call(N):
    """The E4M3 activations lie in one workspace, row-major or K-blocked by the batch: the padding of
    one layout is data of the other, and must not hand an earlier call's NaNs to later cells."""
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[fp8 nan] layouts in turn, N={N}", flush=True)
    mech = chemgen.make_mechanism("ch4")
    K = mech.K
    T, p, Y = (to_dev(x, dev) for x in chemgen.make_states(mech, "ch4", N=N, seed=910))
    m = P.AnnModel(K + 2, K, (1600, 800, 400), seed=5)
    m.fit_norm(T, p, Y, (Y * 1.01).contiguous(), lam=0.1, dt_model=1e-5)
    m.quantize_fp8(T[:4096].contiguous(), p[:4096].contiguous(), Y[:, :4096].contiguous())

    def run(n, bad=False):
        t = torch.full_like(T[:n], float("nan")) if bad else T[:n].clone()
        return m.forward(t, p[:n].contiguous(), Y[:, :n].contiguous(), K).cpu().numpy()

    sizes = (N, 6400, 30011, (1 << 17) - 1)
    good = {n: run(n) for n in sizes}
    assert all(np.isfinite(u).all() for u in good.values())
    for a in sizes:
        for b in sizes:
            assert np.isnan(run(a, bad=True)).all()
            np.testing.assert_array_equal(run(b), good[b])

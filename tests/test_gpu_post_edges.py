"""The surrogate's step on cells whose temperature is none: they are flagged and left as they are."""
import numpy as np
import pytest

import chemgen
from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu


# 4, 8, 16 species to a wave
@pytest.mark.parametrize("which", ["h2", "ch4", "wide"])
def test_post_without_temperature(which):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[post edges] {which}", flush=True)
    mech = chemgen.make_mechanism(which)
    K, N = mech.K, 130
    T, p, Y = chemgen.make_states(mech, "h2" if which == "h2" else "ch4", N=N, seed=43)
    m = P.AnnModel(K + 2, K, (64, 32, 32), seed=3)
    m.fit_norm(to_dev(T, dev), to_dev(p, dev), to_dev(Y, dev), to_dev(Y * 1.01, dev), 0.1, 1e-5)
    for i, v in ((0, 0.0), (5, -0.0), (64, 5e-324), (70, 1e-310), (100, np.inf), (N - 1, np.nan)):
        T[i] = v
    bad = [0, 5, 64, 70, 100, N - 1]
    t, y = to_dev(T, dev), to_dev(Y, dev)
    RR = torch.full_like(y, 3.0)
    fl = torch.full((N,), 9, dtype=torch.uint8, device=dev)
    # a margin and a tolerance that leave nothing else to flag
    m.step(P.Mechanism(mech), 1e-5, t, to_dev(p, dev), y, RR=RR, flags=fl, fallback=False,
           residual_tol=1e30, ood_margin=1e30)
    torch.cuda.synchronize()
    fl, RR = fl.cpu().numpy(), RR.cpu().numpy()
    assert (fl[bad] & 2).all()
    np.testing.assert_array_equal(t.cpu().numpy()[bad], T[bad])
    np.testing.assert_array_equal(y.cpu().numpy()[:, bad], Y[:, bad])
    assert (RR[:, bad] == 0.0).all()
    good = np.setdiff1d(np.arange(N), bad)
    assert not fl[good].any() and np.isfinite(RR[:, good]).all()

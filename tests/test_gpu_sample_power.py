"""The sampler's powers outside the range of the short logarithm, the widest species count and the
range reduction's remainders, against the oracle."""
import numpy as np
import pytest

import chemgen
from oracle import hfrd
from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu


# gamma 0.1: every power near 1; 3: |gamma c ln y| on both sides of the bound, in one wave
@pytest.mark.parametrize("which,N,gamma", [("ch4", 257, 3.0), ("wide", 1000, 0.1), ("wide", 70, 3.0),
                                           ("ch4", 131073, 0.1)])
def test_sampler_powers(which, N, gamma):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[sampler powers] {which} N={N} gamma={gamma}", flush=True)
    mech = chemgen.make_mechanism(which)
    n2 = mech.index("N2")
    T, p, Y = chemgen.make_states(mech, "ch4", N=N, seed=818)
    p = p + 100.0 * np.sin(np.arange(N))
    Y[3, ::5] = 1e-310  # denormal
    c, _ = chemgen.hfrd_randoms(mech.K, N, seed=819, mix_fraction=0.0)
    To, po, Yo, keep = P.sample_states(P.Mechanism(mech), mech, to_dev(T, dev), to_dev(p, dev), to_dev(Y, dev),
                                       to_dev(c, dev), gamma=gamma)
    torch.cuda.synchronize()
    Tr, pr, Yr, _ = hfrd.sample(mech, T, p, Y, c, np.full(N, -1.0), None, None, n2, gamma=gamma)
    np.testing.assert_allclose(To.cpu().numpy(), Tr, rtol=1.6e-15, atol=0)
    np.testing.assert_allclose(po.cpu().numpy(), pr, rtol=1.6e-15, atol=0)
    # |d ln y| < 4 costs 4 eps, the general power an ulp, the rescaling's sum a few
    np.testing.assert_allclose(Yo.cpu().numpy(), Yr, rtol=2e-14, atol=1e-300)

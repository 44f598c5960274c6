"""The sampler's powers against 64-bit mantissas: a single power's error, without what the sum of
many species would hide."""
import numpy as np
import pytest

import chemgen
from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.skipif(np.finfo(np.longdouble).nmant < 63, reason="needs an extended type on the host")
@pytest.mark.parametrize("lo,hi", [(-15.0, -9.0), (-4.0, 0.0)])
def test_sampler_power_error(lo, hi):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[sampler accuracy] y = 10^{lo} .. 10^{hi}", flush=True)
    mech = chemgen.make_mechanism("ch4")
    K, N = mech.K, 1 << 17
    rng = np.random.RandomState(11)
    a, b, n2 = mech.index("OH"), mech.index("O2"), mech.index("N2")
    Y = np.zeros((K, N))
    Y[a] = 10.0 ** rng.uniform(lo, hi, N)
    Y[b] = 1.0  # every power of it is 1
    T, p = np.full(N, 1500.0), np.full(N, 101325.0)
    c = rng.uniform(-1.0, 1.0, (K + 3, N))
    _, _, Yo, _ = P.sample_states(P.Mechanism(mech), mech, to_dev(T, dev), to_dev(p, dev), to_dev(Y, dev),
                                  to_dev(c, dev), alpha=0.0, beta=0.0, gamma=0.1)
    torch.cuda.synchronize()
    x = (1.0 + 0.1 * c[3 + a]).astype(np.longdouble)
    v = np.exp(x * np.log(Y[a].astype(np.longdouble)))
    ref = v / (1 + v)
    err = np.abs(Yo.cpu().numpy()[a] - ref) / ref * 2.0 ** 53
    print(f"  error in units of 2^-53: mean {float(err.mean()):.3f} max {float(err.max()):.3f}", flush=True)
    # one ulp of the power (two units), and a rounding each of the sum, the quotient and the product
    assert err.max() <= 5.001
    assert np.all(Yo.cpu().numpy()[n2] == 0.0)

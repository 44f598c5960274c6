"""chem_rates on states outside any flame's: the limits that the formulas have there (zero, infinity,
NaN), as the oracle's library functions give them."""
import numpy as np
import pytest

import chemgen
import oracle
from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu


# the lane-group kernel's two group widths, and the kernel with one cell per lane
@pytest.mark.parametrize("which", ["h2", "ch4", "wide"])
@pytest.mark.parametrize("N", [13, 8192])
def test_rates_limits(which, N):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[rates limits] {which} N={N}", flush=True)
    mech = chemgen.make_mechanism(which)
    T, p, Y = chemgen.make_states(mech, "h2" if which == "h2" else "ch4", N=N, seed=41)
    T[1], T[2], T[3], T[4], T[5] = 0.0, np.inf, 5e-324, -300.0, np.nan
    Y[-1, 6] = np.inf  # the inert species: no concentration is left for the others
    p[7] = 0.0
    om = oracle.OracleMech(mech)
    with np.errstate(all="ignore"):
        w_o, _, kf_o, kr_o = oracle.chem_rates(om, T, p, Y, want_k=True)
    gm = P.Mechanism(mech)
    args = gm, to_dev(T, dev), to_dev(p, dev), to_dev(Y, dev)
    out = P.chem_rates(*args, kfkr=True)
    one = P.chem_rates(*args)
    torch.cuda.synchronize()
    w = out["wdot"].cpu().numpy()
    np.testing.assert_array_equal(one["wdot"].cpu().numpy(), w)
    # rtol: as over the ordinary states
    np.testing.assert_allclose(out["kf"].cpu().numpy(), kf_o, rtol=1e-12, atol=0)
    fin = [i for i in range(N) if i != 3]  # k_r at a subnormal T: a difference of infinities
    np.testing.assert_allclose(out["kr"].cpu().numpy()[:, fin], kr_o[:, fin], rtol=1e-12, atol=0)
    assert np.isnan(w[:, 1:6]).sum() == np.isnan(w_o[:, 1:6]).sum()
    for i in (6, 7):  # nothing reacts: zero, or NaN of 0 * inf
        np.testing.assert_array_equal(w[:, i], w_o[:, i])

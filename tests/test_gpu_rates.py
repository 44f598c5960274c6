"""chem_rates on batches large enough for one cell per lane, against the oracle."""
import dataclasses

import numpy as np
import pytest

import chemgen
import oracle
from gpu_util import need_gpu, to_dev, one_way_scale

pytestmark = pytest.mark.gpu


# 8191 | 8192: the last size of the lane-group kernel and the first of this one; a last block of
# one cell and of all but one; padded rows
@pytest.mark.parametrize("which,N,pad", [("ch4", 8191, 0), ("ch4", 8192, 0), ("ch4", 8193, 3), ("ch4", 10239, 0),
                                         ("h2", 8257, 1), ("wide", 8200, 0)])
def test_rates_cells(which, N, pad):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[rates cells] {which} N={N} pad={pad}", flush=True)
    mech = chemgen.make_mechanism(which)
    T, p, Y = chemgen.make_states(mech, "ch4" if which == "wide" else which, N=N, seed=303)
    T[5], T[6] = 1000.0, np.nextafter(1000.0, 2000.0)  # either side of T_mid in one wave
    om = oracle.OracleMech(mech)
    Yd = torch.full((mech.K, N + pad), float("nan"), dtype=torch.float64, device=dev)
    Yd[:, :N] = to_dev(Y, dev)
    gm = P.Mechanism(mech)
    out = P.chem_rates(gm, to_dev(T, dev), to_dev(p, dev), Yd, kfkr=True)
    one = P.chem_rates(gm, to_dev(T, dev), to_dev(p, dev), Yd, dTdt=False)
    torch.cuda.synchronize()
    assert torch.equal(one["wdot"], out["wdot"])
    w_o, dT_o, kf_o, kr_o = oracle.chem_rates(om, T, p, Y, want_k=True)
    # an exponent x carries a rounding error of |x| eps, |x| < 1000: 2.2e-13
    np.testing.assert_allclose(out["kf"].cpu().numpy(), kf_o, rtol=1e-12, atol=0)
    np.testing.assert_allclose(out["kr"].cpu().numpy(), kr_o, rtol=1e-12, atol=0)
    sc = one_way_scale(mech, T, p, Y, kf_o, kr_o)
    w_g = out["wdot"].cpu().numpy()
    assert np.all(np.abs(w_g - w_o) <= 1e-12 * sc[None, :] * 4 + 1e-300)
    RG = 8.314462618
    idx = np.arange(0, N, 61)
    hmax = np.array([np.abs(oracle.thermo(om, t)[1]).max() * RG * t for t in T[idx]])
    rho = p[idx] / (RG * T[idx] * (Y[:, idx] / mech.W[:, None]).sum(axis=0))
    cp = np.array([np.sum(Y[:, i] * RG * oracle.thermo(om, T[i])[0] / mech.W) for i in idx])
    err = np.abs(out["dTdt"].cpu().numpy() - dT_o)[idx]
    assert np.all(err <= 1e-12 * mech.R * hmax * sc[idx] * 4 / (rho * cp) + 1e-300)


def test_rates_cells_no_reactions():
    """A mechanism without reactions has zero rates."""
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    m = chemgen.make_mechanism("h2")
    none = dataclasses.replace(m, rsp=m.rsp[:0], rnu=m.rnu[:0], A=m.A[:0], b=m.b[:0], Ea=m.Ea[:0])
    T, p, Y = chemgen.make_states(m, "h2", N=8200, seed=5)
    out = P.chem_rates(P.Mechanism(none), to_dev(T, dev), to_dev(p, dev), to_dev(Y, dev))
    torch.cuda.synchronize()
    assert not out["wdot"].any() and not out["dTdt"].any()

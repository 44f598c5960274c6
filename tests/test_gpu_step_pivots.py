"""The integrator's elimination: pivots off the diagonal (the search's path) and the edges of its
lane layouts, against the oracle."""
import dataclasses

import numpy as np
import pytest

import chemgen
import oracle
from gpu_util import need_gpu, to_dev, compare_state

pytestmark = pytest.mark.gpu


def _shifted(mech, shift):
    """The same chemistry with another enthalpy reference per element (J/mol over R): every reaction's
    enthalpy stays, the order of the species by enthalpy per mass does not."""
    d = mech.comp @ np.array([shift.get(e, 0.0) for e in mech.elements])
    nasa = mech.nasa.copy()
    nasa[:, 8] += d
    nasa[:, 15] += d
    return dataclasses.replace(mech, nasa=nasa)


def _restricted(mech, K):
    """K of the species (those of the mixture first) and the reactions among them."""
    need = [mech.index(s) for s in ("CH4", "O2", "N2", "CO2", "CO", "H2O", "H2", "H", "OH", "O")]
    keep = sorted(need + [k for k in range(mech.K) if k not in need][:K - len(need)])
    new = {k: i for i, k in enumerate(keep)}
    rs = [r for r in range(mech.R) if all(s < 0 or s in new for s in mech.rsp[r])]
    rsp = np.array([[new.get(int(s), -1) for s in mech.rsp[r]] for r in rs], dtype=np.int32)
    return dataclasses.replace(mech, species=[mech.species[k] for k in keep], comp=mech.comp[keep], W=mech.W[keep],
                               nasa=mech.nasa[keep], rsp=rsp, rnu=mech.rnu[rs], A=mech.A[rs], b=mech.b[rs],
                               Ea=mech.Ea[rs], hf298=mech.hf298[keep], s298=mech.s298[keep],
                               radical=mech.radical[keep])


def _check(mech, cfg, N, dt, seed, lanes=0):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    om = oracle.OracleMech(mech)
    T, p, Y = chemgen.make_states(mech, cfg, N=N, seed=seed)
    gm = P.Mechanism(mech)
    if lanes:
        P.chem_set_tuning(gm, lanes_per_cell=lanes)
    Td, pd, Yd = to_dev(T, dev), to_dev(p, dev), to_dev(Y, dev)
    st = torch.zeros((3, N), dtype=torch.int32, device=dev)
    P.chem_step(gm, dt, Td, pd, Yd, stats=st)
    torch.cuda.synchronize()
    o = oracle.chem_step(om, dt, T, p, Y)
    assert np.array_equal(st.cpu().numpy(), o["stats"])
    res = compare_state(Td.cpu().numpy(), Yd.cpu().numpy(), o["T"], o["Y"])
    assert res["ok"], res


# in a third to a half of these attempts the diagonal is not the largest entry of some column
@pytest.mark.parametrize("which,shift,dt,N", [("ch4", {"O": 1e5}, 1e-4, 65), ("ch4", {"H": -1e5}, 1e-4, 33),
                                              ("h2", {"H": 3e4, "O": -1e5}, 1e-2, 67), ("h2", {}, 1e-2, 5)])
def test_step_pivots_off_diagonal(which, shift, dt, N):
    print(f"[step pivots] {which} {shift} dt={dt}", flush=True)
    _check(_shifted(chemgen.make_mechanism(which), shift), which, N, dt, 707)


# n = K + 1 at the ends of the 16- and 32-lane layouts and just past them
@pytest.mark.parametrize("K", [12, 14, 15, 16, 19, 31, 32])
def test_step_layout_edges(K):
    print(f"[step layout] K={K}", flush=True)
    _check(_restricted(chemgen.make_mechanism("wide"), K), "ch4", 37, 1e-5, 708)


@pytest.mark.parametrize("which,lanes", [("h2", 32), ("h2", 64), ("ch4", 64)])
def test_step_wider_groups(which, lanes):
    print(f"[step lanes] {which} {lanes}", flush=True)
    _check(chemgen.make_mechanism(which), which, 41, 1e-6, 709, lanes=lanes)

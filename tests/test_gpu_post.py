"""Post-processing of the surrogate (projection, temperature, rates) over the sizes
its kernel is compiled for, against the oracle on the same network output."""
import dataclasses

import numpy as np
import pytest

import chemgen
import oracle
from oracle import ann as oann
from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu


# 9, 30, 44 species: 4, 8, 16 to a wave; up to four elements and up to eight; blocks of
# 64 cells; padded rows
@pytest.mark.parametrize("which,extra,N,pad", [("h2", 0, 65, 3), ("ch4", 0, 1, 0), ("ch4", 0, 200, 5),
                                               ("ch4", 4, 127, 0), ("h2", 2, 64, 0),
                                               ("wide", 0, 129, 0), ("wide", 3, 63, 1)])
def test_post(which, extra, N, pad):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[post] {which} +{extra} elements N={N} pad={pad}", flush=True)
    mech = chemgen.make_mechanism(which)
    rng = np.random.default_rng(11 + N)
    if extra:  # further conserved quantities, independent of the elements (and no reactions,
        # which would not conserve them)
        mech = dataclasses.replace(
            mech, rsp=mech.rsp[:0], rnu=mech.rnu[:0], A=mech.A[:0], b=mech.b[:0], Ea=mech.Ea[:0],
            elements=mech.elements + [f"X{i}" for i in range(extra)],
            comp=np.concatenate([mech.comp, rng.integers(0, 3, (mech.K, extra))],
                                axis=1).astype(np.int32),
            awt=np.concatenate([mech.awt, np.full(extra, 0.01)]))
    K = mech.K
    om = oracle.OracleMech(mech)
    gm = P.Mechanism(mech)
    T, p, Y = chemgen.make_states(mech, "ch4" if which == "wide" else which, N=N, seed=19)
    T[0] = 1000.0  # T_mid
    feat = oann.features(T, p, Y)
    f32 = lambda a: np.asarray(a, np.float32)
    sd = f32(10.0 ** rng.uniform(-6, -3, K))
    mu = f32(sd * rng.uniform(-0.5, 0.5, K))
    lo, hi = f32(feat.min(axis=1) - 1.0), f32(feat.max(axis=1) + 1.0)
    if N > 2:
        lo[0] = np.sort(T)[1]  # the coldest cell lies outside
        hi[0] = T.max()
    m = P.AnnModel(K + 2, K, (64, 32, 32), seed=5)
    m.set_norm(0.1, 1e-5, feat.mean(axis=1), feat.std(axis=1) + 1e-3, lo, hi, mu, sd)

    def run(tol):
        t, q = to_dev(T, dev), to_dev(p, dev)
        y = torch.full((K, N + pad), 7.0, dtype=torch.float64, device=dev)
        y[:, :N] = to_dev(Y, dev)
        rr = torch.full_like(y, 3.0)
        fl = torch.full((N,), 9, dtype=torch.uint8, device=dev)
        nfb = torch.full((1,), 77, dtype=torch.int64, device=dev)
        m.step(gm, 1e-5, t, q, y, RR=rr, flags=fl, n_fallback=nfb, fallback=False, residual_tol=tol)
        torch.cuda.synchronize()
        assert pad == 0 or (float(y[:, N:].min()) == 7.0 and float(rr[:, N:].max()) == 3.0)
        fl = fl.cpu().numpy()
        assert int(nfb.item()) == np.count_nonzero(fl)
        return t.cpu().numpy(), y[:, :N].cpu().numpy(), rr[:, :N].cpu().numpy(), fl

    U = m.forward(to_dev(T, dev), to_dev(p, dev), to_dev(Y, dev), K).cpu().numpy().astype(np.float64)
    sd64, mu64 = sd.astype(np.float64), mu.astype(np.float64)
    kw = dict(lo=lo.astype(np.float64), hi=hi.astype(np.float64), margin=0.05)
    o = oann.post(om, T, p, Y, U.T, mu64, sd64, 1e-5, residual_tol=1e9, **kw)
    Tg, Yg, RRg, fg = run(1e9)
    np.testing.assert_array_equal(fg, o["flags"])
    ok = fg == 0
    assert ok.sum() >= max(1, N - 2)
    # dY' = sd u + mu is formed in FP32 (two roundings), the rest in FP64; the projection
    # maps an error e of it to (I - D M^T A^-1 M) e, whose gain is taken from the matrices
    M = oann.element_mass_matrix(mech)
    for i in np.flatnonzero(ok):
        yp = np.maximum(o["Yp"][:, i], 0.0)
        d = sd64 ** 2 * (yp + 1e-10) / (yp + sd64)
        G = np.eye(K) - d[:, None] * (M.T @ np.linalg.solve((M * d) @ M.T, M))
        e = 2.0 ** -23 * (np.abs(U[i] * sd64) + np.abs(mu64))
        cond = np.linalg.cond((M * d) @ M.T)
        bound = np.abs(G) @ e + 2.0 ** -52 * (8 * np.abs(Y[:, i]) + cond * np.abs(o["Yp"][:, i] - Y[:, i]).max())
        err = np.abs(Yg[:, i] - o["Y"][:, i])
        assert np.all(err <= bound), (i, (err / bound).max())
        assert np.all(np.abs(RRg[:, i] - o["RR"][:, i]) <= o["rho0"][i] / 1e-5 * bound
                      + 1e-12 * np.abs(o["RR"][:, i]))
    np.testing.assert_allclose(Tg[ok], o["T"][ok], rtol=1e-6)
    np.testing.assert_array_equal(Yg[:, ~ok], Y[:, ~ok])
    np.testing.assert_array_equal(Tg[~ok], T[~ok])
    assert np.all(RRg[:, ~ok] == 0)
    # a tolerance that splits the cells
    res = np.maximum(o["residual"], o["residual_raw"])
    tol = float(np.median(res)) * 1.03
    _, _, _, fg = run(tol)
    want = o["flags"] | np.where(res > tol, 2, 0)
    clear = np.abs(res - tol) > 0.01 * tol
    np.testing.assert_array_equal(fg[clear], want[clear])


def test_post_non_finite():
    """Cells whose state is not finite are flagged and left as they are; their
    neighbours are not affected."""
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print("[post non-finite]", flush=True)
    mech = chemgen.make_mechanism("ch4")
    K, N = mech.K, 70
    gm = P.Mechanism(mech)
    T, p, Y = chemgen.make_states(mech, "ch4", N=N, seed=23)
    m = P.AnnModel(K + 2, K, (64, 32, 32), seed=6)
    feat = oann.features(T, p, Y)
    m.set_norm(0.1, 1e-5, feat.mean(axis=1), feat.std(axis=1) + 1e-3, feat.min(axis=1) - 1,
               feat.max(axis=1) + 1, np.zeros(K), np.full(K, 1e-5))

    def run(T, Y):
        t, y = to_dev(T, dev), to_dev(Y, dev)
        fl = torch.zeros(N, dtype=torch.uint8, device=dev)
        m.step(gm, 1e-5, t, to_dev(p, dev), y, flags=fl, fallback=False, residual_tol=1e9)
        torch.cuda.synchronize()
        return t.cpu().numpy(), y.cpu().numpy(), fl.cpu().numpy()

    t0, y0, f0 = run(T, Y)
    assert not f0.any()
    T2, Y2 = T.copy(), Y.copy()
    T2[1], T2[66], T2[5] = np.nan, np.inf, -np.inf
    Y2[3, 2], Y2[4, 67], Y2[29, 7] = np.nan, np.inf, -np.inf
    bad = np.zeros(N, bool)
    bad[[1, 66, 5, 2, 67, 7]] = True
    t, y, f = run(T2, Y2)
    assert np.all(f[bad] != 0) and not f[~bad].any()
    np.testing.assert_array_equal(t[bad], T2[bad])
    np.testing.assert_array_equal(y[:, bad], Y2[:, bad])
    np.testing.assert_array_equal(t[~bad], t0[~bad])
    np.testing.assert_array_equal(y[:, ~bad], y0[:, ~bad])

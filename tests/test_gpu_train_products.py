"""The products of a training step at the edges of their tiles and splits: gradients
against the oracle on the same data."""
import numpy as np
import pytest

import chemgen
from oracle import ann as oann
from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu


# one 32-row K-step; row tiles of 64 and 96 that end inside; K ranges that do not divide; sides of
# 32 (padded from less), not multiples of 64 or 160, and of both tilings
@pytest.mark.parametrize("hid,B", [((64, 32, 32), 32), ((96, 224, 64), 96), ((1600, 800, 400), 32),
                                   ((1600, 800, 400), 672), ((1600, 800, 400), 2080),
                                   ((1024, 1040, 48), 3104), ((480, 960, 1280), 5152)])
def test_gradients(hid, B):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[train products] {hid} B={B}", flush=True)
    mech = chemgen.make_mechanism("h2")
    K = mech.K
    T, p, Y0 = chemgen.make_states(mech, "h2", N=B, seed=B)
    rng = np.random.default_rng(B)
    Y1 = Y0 * (1 + 0.01 * rng.standard_normal(Y0.shape))
    sizes = [K + 2, *hid, K]
    f32 = lambda a: np.asarray(a, np.float32).astype(np.float64)
    params = [(f32(W), f32(b + 0.1 * rng.standard_normal(b.shape))) for W, b in
              oann.init_params(sizes, seed=13)]
    feat, tgt = oann.features(T, p, Y0), oann.targets(Y0, Y1)
    mi, si = oann.zstats(feat)
    mo, so = oann.zstats(tgt)
    m = P.AnnModel(K + 2, K, hid, seed=1)
    for l, (W, b) in enumerate(params):
        m.set_layer(l, W, b)
    m.set_norm(0.1, 1e-5, mi, si, feat.min(axis=1), feat.max(axis=1), mo, so)
    X = ((feat - f32(mi)[:, None]) / f32(si)[:, None]).T
    tz = ((tgt - f32(mo)[:, None]) / f32(so)[:, None]).T
    grads, loss_o = oann.backward(params, X, tz, prec="bf16")
    loss = torch.zeros(1, dtype=torch.float32, device=dev)
    args = [to_dev(a, dev) for a in (T, p, Y0, Y1)]
    first = None
    for rep in range(2):
        m.train_step(*args, loss, lr=0.0)
        torch.cuda.synchronize()
        got = [m.get_grad(l, (sizes[l + 1], sizes[l])) for l in range(4)]
        if first is not None:  # the sums are in a fixed order
            for a, b in zip(first, got):
                assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        first = got
    assert abs(loss.item() - loss_o) <= 1e-3 * loss_o
    # the bound of the gradient tests: signs of the L1 loss that BF16 rounding flips
    for l in range(4):
        for a, b in ((got[l][0], grads[l][0]), (got[l][1], grads[l][1])):
            rel = np.linalg.norm(a - b) / np.linalg.norm(b)
            print(f"  layer {l} rel {rel:.2e}", flush=True)
            assert rel <= 1e-2


# up to 32 species and up to 63; whole blocks of 64 samples and not; gathered and in order
@pytest.mark.parametrize("which,B,phys", [("h2", 32, True), ("h2", 192, False), ("wide", 96, True),
                                          ("wide", 160, False), ("ch4", 672, True)])
def test_output_gradient(which, B, phys):
    import torch
    import oracle
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[output gradient] {which} B={B} physics={phys}", flush=True)
    mech = chemgen.make_mechanism(which)
    om, gm, K = oracle.OracleMech(mech), P.Mechanism(mech), mech.K
    T, p, Y0 = chemgen.make_states(mech, "ch4" if which == "wide" else which, N=B, seed=B + 1)
    rng = np.random.default_rng(B)
    Y1 = Y0 * (1 + 0.01 * rng.standard_normal(Y0.shape))
    T1 = T + rng.uniform(-300, 300, B)
    f32 = lambda a: np.asarray(a, np.float32).astype(np.float64)
    feat, tgt = oann.features(T, p, Y0), oann.targets(Y0, Y1)
    mi, si = oann.zstats(feat)
    mo, so = oann.zstats(tgt)
    m = P.AnnModel(K + 2, K, (64, 64, 32), seed=2)
    m.set_norm(0.1, 1e-5, mi, si, feat.min(axis=1), feat.max(axis=1), mo, so)
    w = (0.3, 0.2, 0.1) if phys else (0.0, 0.0, 0.0)
    loss = torch.zeros(1, dtype=torch.float32, device=dev)
    terms = torch.zeros(3, dtype=torch.float32, device=dev)
    kw = dict(mech=gm, w_phys=w, terms=terms) if phys else {}
    # gathered from a larger set in another order
    N = B + 37
    order = rng.permutation(N)[:B]
    def spread(a):
        out = np.full(a.shape[:-1] + (N,), 0.5)
        out[..., order] = a
        return to_dev(out, dev)
    index = torch.from_numpy(order.astype(np.int64)).to(dev)
    if phys:
        kw["T1"] = to_dev(T1, dev)
    m.train_step(*[to_dev(a, dev) for a in (T, p, Y0, Y1)], loss, lr=0.0, **kw)
    torch.cuda.synchronize()
    got = [m.get_grad(l, s) for l, s in ((0, (64, K + 2)), (3, (K, 32)))]
    res = (loss.item(), terms.cpu().numpy())
    if phys:
        kw["T1"] = spread(T1)
    m.train_step(*[spread(a) for a in (T, p, Y0, Y1)], loss, index=index, B=B, lr=0.0, **kw)
    torch.cuda.synchronize()
    for (a, b), s, l in zip(got, ((64, K + 2), (K, 32)), (0, 3)):
        gW, gb = m.get_grad(l, s)
        assert np.array_equal(a, gW) and np.array_equal(b, gb)
    assert loss.item() == res[0] and np.array_equal(terms.cpu().numpy(), res[1])
    # the oracle's gradient on the GPU's own output, which inference may round differently by
    # up to TU: signs that close to zero may go either way
    TU = 2e-2
    U = m.forward(to_dev(T, dev), to_dev(p, dev), to_dev(Y0, dev), K).cpu().numpy().astype(np.float64)
    mu, sd = f32(mo), f32(so)
    tz = ((tgt - mu[:, None]) / sd[:, None]).T
    d = U - tz
    g = np.sign(d) / (B * K)
    slack = 2.0 * (np.abs(d) <= TU) / (B * K)
    total = np.abs(d).mean()
    if phys:
        h1 = oann.species_enthalpy(om, T1)
        h0 = np.repeat(oann.species_enthalpy(om, oann.T_REF_HRR), B, axis=1)
        t, gp = oann.physics_terms(U, tz, mu, sd, h1, h0, w)
        g = g + gp
        assert np.all(np.abs(res[1] - t) <= TU)
        total += float(np.dot(w, t))
        dY, e = U * sd + mu, d * sd
        for wt, a, s in zip(w, (np.ones((B, K)), h1.T, h0.T),
                            (dY.sum(axis=1), (h1.T * e).sum(axis=1), (h0.T * e).sum(axis=1))):
            D = (np.abs(a) * sd).sum(axis=1)
            slack = slack + (2.0 * wt * np.abs(a) * sd / (D[:, None] * B)
                             * (np.abs(s) <= TU * D)[:, None])
    assert abs(res[0] - total) <= TU * (1 + sum(w))
    err = np.abs(got[1][1] - g.sum(axis=0))
    bound = slack.sum(axis=0) + 1e-6 * np.abs(g).sum(axis=0)
    print(f"  bias gradient err/bound {(err / bound).max():.3f}, slack share "
          f"{(slack.sum(axis=0) / np.abs(g).sum(axis=0)).max():.3f}", flush=True)
    assert np.all(err <= bound)

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

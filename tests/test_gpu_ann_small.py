"""Small batches of the surrogate run each layer as its own launch of small
tiles; the arithmetic of a cell is that of the large batches' kernels, so its
output row is the same bit for bit whatever batch it is in."""
import numpy as np
import pytest

import chemgen
from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu

LARGE = 24576  # the first size of the fused kernels


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


@pytest.mark.parametrize("name,hid", [("ch4", (1600, 800, 400)), ("h2", (1600, 800, 400)),
                                      ("ch4", (1600, 1200, 400)), ("ch4", (1600, 400, 64))])
def test_rows_do_not_depend_on_the_batch(dev, name, hid):
    import torch
    import paper_2312_05800_amd as P
    print(f"[ann small] {name} {hid}", flush=True)
    mech = chemgen.make_mechanism(name)
    gm = P.Mechanism(mech)
    K = mech.K
    T, p, Y = (to_dev(x, dev) for x in chemgen.make_states(mech, name, N=LARGE, seed=707))
    m = P.AnnModel(K + 2, K, hid, seed=3)
    # training range from the middle of the batch: some cells lie outside
    m.fit_norm(T[100:9000].contiguous(), p[100:9000].contiguous(), Y[:, 100:9000].contiguous(),
               (Y[:, 100:9000] * 1.01).contiguous(), lam=0.1, dt_model=1e-5)

    def run(n):
        t, q, y = T[:n].clone(), p[:n].clone(), Y[:, :n].clone(memory_format=torch.contiguous_format)
        u = m.forward(t, q, y, K)
        flags = torch.full((n,), 9, dtype=torch.uint8, device=dev)
        m.step(gm, 1e-5, t, q, y, flags=flags, fallback=False)
        torch.cuda.synchronize()
        return u.cpu().numpy(), flags.cpu().numpy() & 1

    u, f = run(LARGE)
    assert np.isfinite(u).all() and np.abs(u).max() > 0 and 0 < f.sum() < LARGE
    for n in (1, 15, 63, 64, 65, 500, 2003, 8003, 16001, LARGE - 1):
        print(f"  n={n}", flush=True)
        un, fn = run(n)
        np.testing.assert_array_equal(un, u[:n])
        np.testing.assert_array_equal(fn, f[:n])


@pytest.mark.parametrize("n", [1, 65, 2003])
def test_padded_rows_and_replays(dev, n):
    """Rows longer than the batch, and a captured step replayed after a weight
    change (its weight layouts follow)."""
    import torch
    import paper_2312_05800_amd as P
    print(f"[ann small graph] n={n}", flush=True)
    mech = chemgen.make_mechanism("ch4")
    gm = P.Mechanism(mech)
    K = mech.K
    T, p, Y = (to_dev(x, dev) for x in chemgen.make_states(mech, "ch4", N=2048, seed=708))
    m = P.AnnModel(K + 2, K, (1600, 800, 400), seed=4)
    m.fit_norm(T, p, Y, (Y * 1.01).contiguous(), lam=0.1, dt_model=1e-5)
    wide = torch.full((K, n + 13), 7.0, dtype=torch.float64, device=dev)
    wide[:, :n] = Y[:, :n]
    t, q = T[:n].clone(), p[:n].clone()
    flags = torch.zeros(n, dtype=torch.uint8, device=dev)
    g = m.step_graph(gm, 1e-5, t, q, wide[:, :n], flags=flags, fallback=False, residual_tol=1.0)
    shape = (1600, K + 2)
    for rep in range(3):
        W, b = m.get_layer(0, shape)
        m.set_layer(0, W * (1.0 - 0.01 * rep), b)
        t2, y2 = T[:n].clone(), Y[:, :n].clone(memory_format=torch.contiguous_format)
        f2 = torch.zeros(n, dtype=torch.uint8, device=dev)
        m.step(gm, 1e-5, t2, q, y2, flags=f2, fallback=False, residual_tol=1.0)
        t.copy_(T[:n])
        wide[:, :n] = Y[:, :n]
        g.launch()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(wide[:, :n].cpu().numpy(), y2.cpu().numpy())
        np.testing.assert_array_equal(t.cpu().numpy(), t2.cpu().numpy())
        np.testing.assert_array_equal(flags.cpu().numpy(), f2.cpu().numpy())
        assert float(wide[:, n:].min()) == 7.0 and float(wide[:, n:].max()) == 7.0

"""Small batches of networks of other widths than 1600-800-400, on the route that runs each layer as
its own launch: the same output rows, bit for bit, as the large batches' kernels."""
import numpy as np
import pytest

import chemgen
from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu

LARGE = 24576  # the first size of the fused kernels


# a second layer of 800 or 1600 takes the route; first layers of one K-step and of the most, third
# layers of one column tile, of remainders and wide
@pytest.mark.parametrize("hid", [(1600, 800, 32), (32, 800, 64), (2048, 1600, 96), (96, 1600, 1280), (64, 800, 208)])
def test_rows_do_not_depend_on_the_batch(hid):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    print(f"[ann small widths] {hid}", flush=True)
    mech = chemgen.make_mechanism("h2")
    K = mech.K
    T, p, Y = (to_dev(x, dev) for x in chemgen.make_states(mech, "h2", N=LARGE, seed=717))
    m = P.AnnModel(K + 2, K, hid, seed=3)
    m.fit_norm(T, p, Y, (Y * 1.01).contiguous(), lam=0.1, dt_model=1e-5)

    def run(n):
        P.profile_enable(True)
        u = m.forward(T[:n].contiguous(), p[:n].contiguous(), Y[:, :n].contiguous(), K)
        torch.cuda.synchronize()
        labels = set(P.profile_read())
        P.profile_enable(False)
        return u.cpu().numpy(), labels

    u, labels = run(LARGE)
    assert "mlp_l12" in labels and "ann_features_l1" not in labels
    assert np.isfinite(u).all() and np.abs(u).max() > 0
    for n in (1, 63, 65, 2003, 8003, LARGE - 1):
        print(f"  n={n}", flush=True)
        un, labels = run(n)
        assert "ann_features_l1" in labels and "mlp_l12" not in labels
        np.testing.assert_array_equal(un, u[:n])

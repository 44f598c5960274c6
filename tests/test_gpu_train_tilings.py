"""The generic tilings of the training products, which only a stored tuning result selects: gradients
of a step with them against the built-in ones (another order of FP32 sums)."""
import numpy as np
import pytest

import chemgen
from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu

B, HID = 2048, (1600, 800, 400)

# tile and K-step of the eleven products (0: built in), splits of the four weight gradients
FORMS = {
    "all 128x128": ([(1, 32)] * 11, (1, 4, 4, 16)),
    "all 128x32": ([(2, 32)] * 11, (16, 16, 16, 16)),
    "all 64x64": ([(3, 32)] * 4 + [(3, 64)] * 4 + [(3, 32)] * 3, (2, 1, 1, 1)),
    "all 128x64": ([(4, 32)] * 4 + [(4, 64)] * 4 + [(4, 32)] * 3, (4, 4, 4, 4)),
    "first data gradient generic": ([(0, 0)] * 8 + [(1, 32), (0, 0), (0, 0)], (16, 4, 4, 16)),
    "first layer generic": ([(3, 32)] + [(0, 0)] * 10, (16, 4, 4, 16)),
    "other ranges": ([(0, 0)] * 11, (1, 1, 2, 8)),
}


@pytest.fixture(scope="module", params=[1, 9], ids=["one network", "ensemble"])
def case(request):
    import torch
    import paper_2312_05800_amd as P
    dev = need_gpu()
    mech = chemgen.make_mechanism("h2")
    K = mech.K
    T, p, Y0 = chemgen.make_states(mech, "h2", N=B, seed=411)
    Y1 = Y0 * (1 + 0.01 * np.random.default_rng(5).standard_normal(Y0.shape))
    args = [to_dev(a, dev) for a in (T, p, Y0, Y1)]
    members = request.param
    shapes = [(HID[0], K + 2), (HID[1], HID[0]), (HID[2], HID[1]), (1 if members > 1 else K, HID[2])]

    def step(line=None, cache=None, monkeypatch=None):
        m = P.AnnModel(K + 2, K, HID, seed=3, members=members)
        m.fit_norm(*args, 0.1, 1e-5)
        if line is not None:
            monkeypatch.setenv("CHEM_AUTOTUNE_CACHE", str(cache))
            cache.write_text(line)
            assert m.autotune_train(B)["products_ms_tuned"] == 0.25  # taken from the file
        loss = torch.zeros(1, dtype=torch.float32, device=dev)
        m.train_step(*args, loss, lr=0.0)
        torch.cuda.synchronize()
        return loss.item(), [m.get_grad(4 * g + l, shapes[l]) for g in range(members) for l in range(4)]

    def key(cache, monkeypatch):
        monkeypatch.setenv("CHEM_AUTOTUNE_CACHE", str(cache))
        P.AnnModel(K + 2, K, HID, seed=3, members=members).autotune_train(B)
        return cache.read_text().split(" = ")[0]
    most = (16, 16, 16, 16) if members == 1 else (16, 2, 8, 16)  # ranges the workspace holds
    return step, key, most, step()


@pytest.mark.parametrize("form", list(FORMS))
def test_generic_tilings(case, form, tmp_path, monkeypatch):
    step, key, most, (loss0, g0) = case
    print(f"[train tilings] {form}", flush=True)
    tiles, splits = FORMS[form]
    line = key(tmp_path / "key", monkeypatch) + " = " + " ".join(f"{t} {b}" for t, b in tiles) + " " + \
        " ".join(str(s) for s in np.minimum(splits, most)) + " 0.5 0.25\n"
    loss, g = step(line, tmp_path / "line", monkeypatch)
    assert loss == loss0  # the forward's sums do not depend on the tiling
    for (a, b), (c, d) in zip(g, g0):
        for x, y in ((a, c), (b, d)):
            rel = np.linalg.norm(x - y) / max(np.linalg.norm(y), 1e-30)
            assert rel <= 1e-5, rel

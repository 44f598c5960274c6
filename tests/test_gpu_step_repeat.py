"""The integrator's repeated elimination (pivots searched for among rows in registers) at the edges
of its lane layouts: mechanisms whose enthalpy reference puts the pivots off the diagonal."""
import pytest

import chemgen
from test_gpu_step_pivots import _check, _restricted, _shifted

pytestmark = pytest.mark.gpu


# n = K + 1 within the 16- and 32-lane layouts, at their ends and just past the first
@pytest.mark.parametrize("K", [12, 14, 15, 16, 19, 31])
def test_step_repeat_edges(K):
    print(f"[step repeat] K={K}", flush=True)
    _check(_restricted(_shifted(chemgen.make_mechanism("wide"), {"O": 1e5}), K), "ch4", 37, 1e-4, 711)

"""The FP64 pair pass on both sides of the lines that choose between teams of
lanes and one lane per particle, where the oracle cannot reach."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_edges import _block

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


@pytest.mark.parametrize("n,cell", [(700000, 1.0005), (700001, 1.0005), (700001, 2.001), (705000, 1.0), (705000, 2.0),
                                    (2000001, 1.0), (3000001, 2.0)])
def test_rebuilding_with_kept_lists_equals_without(n, cell):
    """Steps too long for the cells' room: every stage rebuilds, bit for bit
    as without the flag, above as below the counts where one form of the pass
    gives way to the other."""
    from paper_2608_22269_amd import Simulation
    dx = 0.0105 if n < 1000000 else 0.0075 if n < 2500000 else 0.0065
    case = _block(n, dx=dx, seed=6)
    case = wl.with_params(case, cell_size=cell * case["params"]["h"])
    a = Simulation(wl.with_params(case, keep_lists=True, keep_across_steps=True))
    b = Simulation(case)
    for s in (a, b):
        s.step(1, 2e-4)
    st = a.stats()
    assert st["n_kept"] == 0 and st["n_rebuilt"] == (2 if cell % 1.0 else 0)  # no room: no lists
    for name in ("x", "u", "phi", "dudt", "dphidt", "nnb"):
        assert np.array_equal(a.field(name), b.field(name)), name
    for s in (a, b):
        s.close()

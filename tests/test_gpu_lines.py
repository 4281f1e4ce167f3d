"""The FP64 pair pass on both sides of the lines that choose between teams of
lanes and one lane per particle, where the oracle cannot reach."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_edges import _block
from test_gpu_parity import _flags_all
from test_gpu_team import _same_rates

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


@pytest.mark.parametrize("dim,n", [(2, 35000), (2, 35001), (3, 70000), (3, 70001)])
def test_from_kept_lists(dim, n):
    """Lists built by teams and read by teams or by a lane per particle: two
    steps against the path that searches at every stage, at the bars of the
    kept lists' other tests."""
    from paper_2608_22269_amd import Simulation
    if dim == 3:
        case = _block(n, dx=0.012, seed=1)
    else:
        case = wl.tank2d(dx=0.0037, **_flags_all())
        fluid = np.nonzero(case["kind"] == 0)[0]
        drop = np.isin(np.arange(len(case["kind"])), fluid[np.argsort(case["x"][fluid, 1])[n:]])
        case = dict(case, **{k: case[k][~drop] for k in ("x", "u", "phi", "kind", "normal")})
        case = wl.random_velocity(case, 0.02, 3)
    case = wl.with_params(case, cell_size=2.1 * case["params"]["h"])
    keep, plain = Simulation(wl.with_params(case, keep_lists=True)), Simulation(case)
    assert keep.nf == n
    for s in (keep, plain):
        s.step(2)
    assert keep.stats()["n_kept"] == 2
    _same_rates(keep, plain)
    assert np.abs(keep.field("x") - plain.field("x")).max() <= 1e-12
    for s in (keep, plain):
        s.close()


@pytest.mark.parametrize("n", [2000000, 2000001])
def test_plain_search_over_cells_of_h(n):
    """Teams or a lane per particle over cells of h against teams over cells
    of 2h, whose windows, lists and orders of summation differ."""
    from paper_2608_22269_amd import Simulation
    case = _block(n, dx=0.0075, seed=4)
    h = case["params"]["h"]
    a, b = (Simulation(wl.with_params(case, cell_size=c * h)) for c in (1.0, 2.0))
    for s in (a, b):
        s.eval_rates()
    _same_rates(a, b)
    for s in (a, b):
        s.close()

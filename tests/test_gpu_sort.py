"""The sort at the edges of its dispatch: the particle count up to which the
hash adds up the scan's tiles (12,000), the key count up to which the scan
works from plain tile sums (4,096 tiles of 1,024 keys), and particles given in
an order that has nothing to do with space (the places inside the cells come
from the original indices).  Against the oracle at the parity bars."""
import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_edges import _block
from test_gpu_parity import compare_rates

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


def _shuffled(case, seed):
    order = np.random.default_rng(seed).permutation(len(case["kind"]))
    return dict(case, **{k: case[k][order] for k in ("x", "u", "phi", "kind", "normal")})


@pytest.mark.parametrize("n,hi", [(12000, 1.0), (12001, 1.0), (32769, 1.0), (500, 1.0), (500, 8.15), (500, 8.37)])
def test_sort_dispatch(n, hi):
    """hi: extent of the domain; at dx = 0.02 (cells of 0.052) 1 m makes 12
    tiles of sort keys, 8.15 m 157 x 160 x 160 keys (3,925 tiles) and 8.37 m
    161 x 168 x 168 (4,438)."""
    from paper_2608_22269_amd import Simulation
    case = _shuffled(_block(n, dx=0.02, seed=n), n + 1)
    case["params"] = dict(case["params"], domain_hi=[hi] * 3)
    sim = Simulation(case)
    for _ in range(3):  # the scratch a sort leaves cleared serves the next one
        sim.build_cells()
    assert np.array_equal(sim.field("cell"), oracle.cells(case["params"], case["x"])[0])
    sim.eval_rates()
    compare_rates(sim, case, oracle.eval_rates(case))
    sim.step(2)
    out = oracle.step(case, 2)
    assert np.abs(sim.field("x") - out["x"]).max() <= 1e-12
    assert np.abs(sim.field("u") - out["u"]).max() <= 1e-12 * np.abs(out["u"]).max()
    sim.close()


def test_many_particles_in_one_cell():
    """Cells of 2h = 12 dx hold some 1,700 particles: beyond the rank by
    original index (1,024), where the order inside a cell is that of arrival;
    neighbour counts and rates are those of the oracle all the same."""
    from paper_2608_22269_amd import Simulation
    case = _shuffled(_block(1728, dx=0.02, seed=3), 4)
    h = 6.0 * 0.02
    case["params"] = dict(case["params"], h=h, cell_size=2.0 * h)
    sim = Simulation(case)
    sim.eval_rates()
    ref = oracle.eval_rates(case)
    assert np.array_equal(sim.field("nnb"), ref["nnb"])
    scale = max(9.81, np.abs(ref["acc"]).max())
    assert np.abs(sim.field("dudt") - ref["acc"]).max() <= 1e-12 * scale
    sim.close()

"""The statistics that the workgroups add to 64 copies of the counters: with
fewer workgroups than copies, one per copy, and more, the totals equal what
the exported fields count, exactly, and U_max is the largest velocity."""
import numpy as np
import pytest

from test_gpu_edges import _block

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [1, 60, 64 * 256, 64 * 256 + 1, 150 * 256])
def test_counters_equal_the_fields(n, precision):
    from paper_2608_22269_amd import Simulation
    case = _block(n, dx=0.02, seed=n)
    case["params"] = dict(case["params"], precision=precision)
    sim = Simulation(case)
    for _ in range(2):  # cleared between right-hand sides
        sim.eval_rates()
        st = sim.stats()
        assert st["n_fs"] == sim.field("fs").sum()
        assert st["n_cons"] == sim.field("tic").sum()
        assert st["pairs"] == sim.field("nnb").sum(dtype=np.int64)
    sim.step(1)
    u = sim.field("u")
    sim.eval_rates()
    umax = np.sqrt((u[case["kind"] == 0] ** 2).sum(axis=1).max())
    assert sim.stats()["umax"] == pytest.approx(umax, rel=1e-14 if precision == "fp64" else 1e-6)
    sim.close()

"""The FP64 pair pass at the edges of its dispatch: teams of 8 lanes per
particle (blocks of 32 particles) up to 3,000,000 particles in 3D and 120,000
in 2D, 700,000 and 120,000 where it builds lists, 130,000 and 40,000 from kept
lists, one lane per particle beyond; over
cells of 2h in 3D the rows are tested in place, else listed.  Against the
oracle at the parity bars; the changeovers that the oracle cannot reach
against the same right-hand side over other cells or without lists."""
import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_edges import _block
from test_gpu_parity import _flags_all, compare_rates

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


def _sim(case):
    from paper_2608_22269_amd import Simulation
    return Simulation(case)


@pytest.mark.parametrize("cell", [2.0, 1.0, 0.7])
@pytest.mark.parametrize("n", [1, 7, 31, 32, 33, 700])
def test_block_edges(n, cell):
    case = _block(n, dx=0.02, seed=n)
    sim = _sim(wl.with_params(case, cell_size=cell * case["params"]["h"]))
    sim.eval_rates()
    compare_rates(sim, case, oracle.eval_rates(case))
    sim.close()


@pytest.mark.parametrize("ratio,n", [(2.6, 1000), (4.0, 1728)])
@pytest.mark.parametrize("cell", [2.0, 1.0])
def test_many_neighbours(ratio, n, cell):
    """h / dx = 2.6 and 4: up to some 590 and 1,728 neighbours, so that the
    list of 160 is emptied several times, and beyond the 256 kept ones."""
    case = _block(n, dx=0.02, seed=5)
    h = ratio * 0.02
    case["params"] = dict(case["params"], h=h, cell_size=cell * h)
    sim = _sim(case)
    sim.eval_rates()
    ref = oracle.eval_rates(case)
    assert np.array_equal(sim.field("nnb"), ref["nnb"])
    scale = max(9.81, np.abs(ref["acc"]).max())
    assert np.abs(sim.field("dudt") - ref["acc"]).max() <= 1e-12 * scale
    keep = _sim(wl.with_params(case, cell_size=1.05 * cell * h, keep_lists=True))
    plain = _sim(wl.with_params(case, cell_size=1.05 * cell * h))
    keep.step(2)
    plain.step(2)
    assert keep.stats()["n_kept"] == 0  # over 256 candidates: every stage searches
    assert np.array_equal(keep.field("u"), plain.field("u"))
    for s in (sim, keep, plain):
        s.close()


def test_other_shifting_exponent():
    case = _block(300, dx=0.02, seed=2)
    case["params"] = dict(case["params"], pst_n=3.0)
    for cell in (2.0, 1.0):
        sim = _sim(wl.with_params(case, cell_size=cell * case["params"]["h"]))
        sim.eval_rates()
        compare_rates(sim, case, oracle.eval_rates(case))
        sim.close()


def _same_rates(a, b):
    assert np.array_equal(a.field("nnb"), b.field("nnb"))
    for f in ("dudt", "dphidt", "lambda", "delta_u"):
        x, y = a.field(f), b.field(f)
        assert np.abs(x - y).max() <= 1e-12 * max(9.81, np.abs(y).max()), f


@pytest.mark.parametrize("n", [119999, 120001])
def test_changeover_2d(n):
    """Around 120,000 particles in 2D, every particle against the oracle."""
    case = wl.tank2d(dx=0.002, **_flags_all())
    fluid = np.nonzero(case["kind"] == 0)[0]
    assert len(fluid) > n
    drop = np.isin(np.arange(len(case["kind"])), fluid[np.argsort(case["x"][fluid, 1])[n:]])
    case = dict(case, **{k: case[k][~drop] for k in ("x", "u", "phi", "kind", "normal")})
    case = wl.random_velocity(case, 0.05, 3)
    sim = _sim(case)
    assert sim.nf == n
    sim.eval_rates()
    compare_rates(sim, case, oracle.eval_rates(case))
    sim.close()


@pytest.mark.parametrize("dim,n", [(2, 39999), (2, 40001), (3, 129999), (3, 130001), (3, 700000), (3, 700001)])
def test_changeover_from_kept_lists(dim, n):
    """Lists built and read by teams, built by teams and read by a lane per
    particle, and both by a lane: two steps against the path that searches at
    every stage."""
    if dim == 3:
        case = _block(n, dx=0.012 if n < 200000 else 0.0105, seed=1)
    else:
        case = wl.tank2d(dx=0.0035, **_flags_all())
        fluid = np.nonzero(case["kind"] == 0)[0]
        assert len(fluid) > n
        drop = np.isin(np.arange(len(case["kind"])), fluid[np.argsort(case["x"][fluid, 1])[n:]])
        case = dict(case, **{k: case[k][~drop] for k in ("x", "u", "phi", "kind", "normal")})
        case = wl.random_velocity(case, 0.02, 3)
    case = wl.with_params(case, cell_size=(2.1 if n < 200000 else 1.03) * case["params"]["h"])
    keep, plain = _sim(wl.with_params(case, keep_lists=True)), _sim(case)
    assert keep.nf == n
    for s in (keep, plain):
        s.step(2)
    assert keep.stats()["n_kept"] == 2
    _same_rates(keep, plain)
    assert np.abs(keep.field("x") - plain.field("x")).max() <= 1e-12
    for s in (keep, plain):
        s.close()


@pytest.mark.parametrize("n", [3000000, 3000001])
def test_changeover_3d(n):
    """Around 3,000,000 particles: cells of h against cells of 2h, whose
    windows, lists and orders of summation differ."""
    case = _block(n, dx=0.0065, seed=4)
    h = case["params"]["h"]
    a, b = _sim(wl.with_params(case, cell_size=h)), _sim(wl.with_params(case, cell_size=2.0 * h))
    for s in (a, b):
        s.eval_rates()
    _same_rates(a, b)
    for s in (a, b):
        s.close()

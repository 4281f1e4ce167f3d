"""The wall mirror on both sides of its dispatch (a team of lanes per wall
particle up to 90,000, or 150,000 in the mixed form, one lane beyond) with one, two and three cells
searched on each side: 9, 25 and 49 rows, on a jittered lattice and on a plain
one, whose equidistant sources are told apart by their index.  Against the
oracle at the parity bars (sources exact, values and rates 1e-12)."""
import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_parity import _flags_all, compare_rates

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


@pytest.mark.parametrize("jitter", [0.1, 0.0])
@pytest.mark.parametrize("layers,reach", [(3, 3), (9, 1), (9, 2), (9, 3)])
def test_mirror_dispatch(layers, reach, jitter):
    from paper_2608_22269_amd import Simulation
    case = wl.box3d(0.02, (1.0, 0.9, 0.9), (1.0, 0.9, 0.1), layers=layers, **_flags_all())
    case = wl.random_velocity(wl.jitter(case, jitter, 21) if jitter else case, 0.05, 22)
    case = wl.with_params(case, cell_size=2.0 * case["params"]["h"] / reach)
    nd = (case["kind"] != 0).sum()
    assert nd > 150000 if layers == 9 else nd < 90000
    sim = Simulation(case)
    sim.eval_rates()
    compare_rates(sim, case, oracle.eval_rates(case))
    sim.close()
    if not jitter:
        return
    mixed = wl.with_params(case, precision="mixed")
    sm = Simulation(mixed)
    sm.eval_rates()
    d = case["kind"] != 0
    src = oracle.eval_rates(case)["mir_src"]
    # FP32 distances may swap two nearly equidistant sources
    assert (sm.field("mirror_src")[d] != src[d]).sum() <= 1e-3 * d.sum()
    sm.close()


@pytest.mark.parametrize("nd", [40, 90100])
def test_no_source_at_nan(nd):
    """A particle whose position has become NaN is kept in cell 0 until the
    error is reported; wall particles around that cell, out of reach of any
    fluid, must not take it for their source (a field exported to the device
    does not wait for the error)."""
    import torch
    from paper_2608_22269_amd import Simulation, _lib as L
    dx = 0.01
    rng = np.random.default_rng(3)
    pd = wl.base_params(2, dx, domain_lo=[0.0] * 3, domain_hi=[1.0, 1.0, 0.0], depth=0.1)
    g = np.stack(np.meshgrid(np.arange(10), np.arange(10), indexing="ij"), -1).reshape(-1, 2)
    xf, xd = 0.5 + dx * g, rng.uniform(0.0, 4.0 * pd["h"], (nd, 2))
    phi = np.zeros(100 + nd)
    phi[55] = 800.0 * pd["c0"] ** 2  # its density overflows
    normal = np.zeros((100 + nd, 2))
    normal[100:, 1] = 1.0
    case = {"params": pd, "x": np.concatenate([xf, xd]), "u": np.zeros((100 + nd, 2)), "phi": phi,
            "kind": np.repeat(np.array([0, 1], np.uint8), [100, nd]), "normal": normal, "mass": None, "t": 0.0,
            "meta": {}}
    sim = Simulation(case)
    sim.step(2, dt=1e-4)
    x = torch.zeros((sim.n, 2), dtype=torch.float64, device="cuda")
    src = torch.zeros(sim.n, dtype=torch.int32, device="cuda")
    sim.field_device("x", x)
    sim.field_device("mirror_src", src)
    torch.cuda.synchronize()
    assert torch.isnan(x[:100]).any()
    assert (src[100:] == -1).all()
    with pytest.raises(L.SphError):
        sim.sync()
    sim.close()


def _far_pairs(copies, seed=0):
    """Wall particles 1,000 m (100,000 cells of h) from the origin, where FP32
    positions lie 0.006 cells apart, `copies` on each place.  Each has two
    fluid particles: one in its own row of cells, nearer by a few thousandths
    of a cell or as far as the other, which lies just inside the second row
    above."""
    rng = np.random.default_rng(seed)
    h = 0.01
    pd = wl.base_params(2, h / 1.3, domain_lo=[1000.0, 1000.0, 0.0], domain_hi=[1003.6, 1000.5, 0.0], depth=0.1,
                        precision="mixed")
    pd = dict(pd, h=h, cell_size=h)
    lo = np.array(pd["domain_lo"][:2])
    c = np.stack(np.meshgrid(4 + 6 * np.arange(58), 4 + 6 * np.arange(7), indexing="ij"), -1).reshape(-1, 2)
    d = lo + (c + np.stack([rng.uniform(0.3, 0.7, len(c)), np.full(len(c), 0.5)], 1)) * h
    above = d + np.stack([np.zeros(len(c)), rng.uniform(1.5005, 1.506, len(c))], 1) * h
    beside = d + np.stack([rng.uniform(1.490, 1.504, len(c)), np.zeros(len(c))], 1) * h
    x = np.concatenate([above, beside, np.repeat(d, copies, axis=0)])
    nf, n = 2 * len(c), len(x)
    normal = np.zeros((n, 2))
    normal[nf:, 1] = 1.0
    case = {"params": pd, "x": x, "u": np.zeros((n, 2)), "phi": np.zeros(n),
            "kind": np.repeat(np.array([0, 1], np.uint8), [nf, n - nf]), "normal": normal, "mass": None, "t": 0.0,
            "meta": {}}
    # positions as the library stores them: an FP32 offset in the cell, then
    # FP32; differences and squares of these are exact in FP32
    corner = lo + np.floor((x[:nf] - lo) / h) * h
    stored = (corner + (x[:nf] - corner).astype(np.float32)).astype(np.float32)
    mid = np.abs(np.abs(stored - (corner + (x[:nf] - corner).astype(np.float32))) / np.spacing(stored) - 0.5)
    sure = (mid > 1e-2).all(1)
    sure = sure[:nf // 2] & sure[nf // 2:]
    r2 = ((stored - np.concatenate([d, d]).astype(np.float32)) ** 2).sum(1)
    src = np.where(r2[:nf // 2] <= r2[nf // 2:], np.arange(nf // 2), np.arange(nf // 2, nf))
    return case, np.repeat(src, copies), np.repeat(sure, copies)


@pytest.mark.parametrize("copies", [1, 400])
def test_mixed_mirror_far_from_the_origin(copies):
    """The source is the nearest in FP32 positions (ties: the lower index)
    also where their rounding is far above a thousandth of a cell: a team of
    lanes per wall particle, and one lane."""
    from paper_2608_22269_amd import Simulation
    case, src, sure = _far_pairs(copies)
    nd = len(src)
    assert nd < 90000 if copies == 1 else nd > 150000
    assert sure.mean() > 0.9
    sim = Simulation(case)
    sim.eval_rates()
    got = sim.field("mirror_src")[-nd:]
    assert np.array_equal(got[sure], src[sure])
    sim.close()

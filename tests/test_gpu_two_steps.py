"""Steps taken two at a time (one pass over the grid per pair) against single
steps: bitwise equal, whatever the parity of the counts, and within the FP64
bar of the oracle.  The sizes are ones the two-step pass is chosen for, with
tiles of one column, one row and a short last chunk of planes among them."""
import numpy as np
import pytest

import oracle as O
from paper_1710_02065_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = [
    (19, (193, 73, 121), "f32", 0), (19, (64, 64, 64), "f32", 0),
    (19, (320, 17, 300), "f32", 0), (19, (256, 8, 300), "f32s", 0),
    (19, (193, 73, 121), "f64", 0), (19, (250, 131, 97), "f16s", 0),
    (27, (193, 73, 121), "f32", 0), (27, (193, 73, 121), "f32s", 1),
    (27, (256, 128, 128), "f16s", 0), (27, (193, 73, 121), "f64", 1),
]


def _sim(q, shape, storage, full, seed=3):
    from paper_1710_02065_amd import lbm
    rho, u, p = W.random_state(shape, seed=seed, d=2 if q == 9 else 3)
    sim = lbm.Simulation(lattice=q, shape=shape, storage=storage, tau=0.53, rho0=1.0625,
                         flags=lbm.LBM_FULL_ORDER if full else 0)
    return sim.init(rho * 1.0625, u, p), (rho * 1.0625, u, p)


@pytest.mark.parametrize("q,shape,storage,full", CASES)
def test_pairs_equal_single_steps_bitwise(q, shape, storage, full):
    import torch
    a, _ = _sim(q, shape, storage, full)
    b, _ = _sim(q, shape, storage, full)
    for n in (2, 5, 67):  # a pair, pairs and a single step, graph replays too
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert a.time == b.time
        assert torch.equal(a.populations(), b.populations())
    a.sync()


@pytest.mark.parametrize("q,full", [(19, 0), (27, 0), (27, 1)])
def test_pairs_match_the_oracle_f64(q, full):
    shape = (193, 73, 121)
    sim, (rho, u, p) = _sim(q, shape, "f64", full)
    f = sim.step(4).populations().cpu().numpy()
    sim.sync()
    g = O.Grid(q, *shape, tau=0.53, rho0=1.0625, full_order=bool(full)).init(rho, u, p).step(4)
    assert np.abs(f - g.f).max() <= 1e-12 * np.abs(g.f).max()


def test_instability_in_a_pair_is_reported():
    from paper_1710_02065_amd import lbm
    shape = (64, 64, 64)
    rho, u, p = W.random_state(shape, seed=1, d=3)
    rho[12345] = float("nan")
    sim = lbm.Simulation(lattice=19, shape=shape, storage="f32", tau=0.53).init(rho, u, p)
    sim.step(2)
    with pytest.raises(lbm.LbmError) as e:
        sim.sync()
    assert e.value.code == lbm.LBM_EUNSTABLE


@pytest.mark.parametrize("q,shape,full", [(9, (192, 160, 1), 0), (9, (192, 160, 1), 1),
                                          (19, (32, 32, 32), 0), (19, (193, 73, 41), 0),
                                          (27, (32, 32, 32), 0), (27, (32, 32, 32), 1)])
def test_fp32_mass_does_not_drift(q, shape, full):
    """Rounding must not add mass step after step.  A cell's density changes by
    up to half an ulp of 1 (6e-8, either sign) a step; over 30,000 cells and
    400 steps that averages to 4e-9.  A rest population whose weight is
    rounded differently in the collision and in the moments adds half an ulp of
    it (7e-9 to 1.5e-8) on every step; the bar is 1e-9 a step."""
    sim, _ = _sim(q, shape, "f32", full)
    n = 400
    before = sim.populations().double().sum().item()
    after = sim.step(n).populations().double().sum().item()
    sim.sync()
    assert abs(after - before) / np.prod(shape) <= n * 1e-9

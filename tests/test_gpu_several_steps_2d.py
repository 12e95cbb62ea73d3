"""D2Q9 steps taken two or four in one pass against single steps (bitwise) and
the oracle (FP64 bar): periodic and general grids, tiles of one column or row,
grids barely as wide as the halo, counts that leave one to three steps over,
and batches of uneven step counts."""
import numpy as np
import pytest

import oracle as O
from paper_1710_02065_amd import workloads as W

pytestmark = pytest.mark.gpu

F64_TOL = 1e-12


def _channel(nx, ny, noise):
    U = 0.2 / np.sqrt(3)
    mask = W.cylinder_mask(nx, ny, max(4, ny // 8), nx // 4, ny // 2)
    return dict(tau=0.56, ma=0.2, face_bc=(2, 2, 1, 1, 0, 0),
                sponge_width=(0, max(3, nx // 8), 0, 0, 0, 0), chi_max=0.2, rho_ref=1.0,
                u_ref=(U, 0.0, 0.0), seed=11, inlet_noise=noise), mask


def _setup(kind, nx, ny):
    rho, u, p = W.random_state((nx, ny, 1), seed=nx + ny, d=2)
    if kind == "box":
        return dict(tau=0.55, rho0=0.9375), None, rho * 0.9375, u, p
    if kind == "closed":
        return dict(tau=0.6), W.closed_box_mask(nx, ny), rho, u, p
    if kind == "posts":  # periodic, with SOLID cells on both sides of the wrap
        m = np.zeros(nx * ny, dtype=np.uint8)
        m[[0, nx - 1, (ny - 1) * nx, (ny // 2) * nx + nx // 2]] = W.SOLID
        return dict(tau=0.6), m, rho, u, p
    if kind == "slip":  # free-slip on every side: corners reflect twice
        return dict(tau=0.6, face_bc=(1, 1, 1, 1, 0, 0)), None, rho, u, p
    kw, mask = _channel(nx, ny, 0.02 if kind == "noise" else 0.0)
    return kw, mask, 1 + 0.1 * (rho - 1), 0.1 * u + np.array([[0.1], [0], [0]]), p


def _sim(kind, nx, ny, storage, full):
    from paper_1710_02065_amd import lbm
    kw, mask, rho, u, p = _setup(kind, nx, ny)
    sim = lbm.Simulation(lattice=9, shape=(nx, ny, 1), storage=storage,
                         flags=lbm.LBM_FULL_ORDER if full else 0, **kw)
    return sim.init(rho, u, p, mask)


SHAPES = [("box", 70, 37), ("box", 65, 9), ("box", 4, 4), ("box", 5, 130), ("box", 3, 40),
          ("closed", 66, 17), ("posts", 129, 23), ("slip", 67, 18), ("channel", 200, 90),
          ("noise", 131, 67), ("channel", 1100, 1000)]


@pytest.mark.parametrize("kind,nx,ny", SHAPES)
@pytest.mark.parametrize("storage", ["f64", "f32", "f32s", "f16s"])
def test_fused_steps_equal_single_steps_bitwise(kind, nx, ny, storage):
    import torch
    full = (nx + ny) % 2
    a, b = _sim(kind, nx, ny, storage, full), _sim(kind, nx, ny, storage, full)
    for n in (2, 3, 4, 7, 70):
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert a.time == b.time
        assert torch.equal(a.populations(), b.populations()), n
    a.sync()


@pytest.mark.parametrize("kind,nx,ny", [("box", 130, 21), ("closed", 66, 17), ("posts", 129, 23),
                                        ("slip", 67, 18), ("noise", 131, 67)])
def test_fused_steps_match_the_oracle_f64(kind, nx, ny):
    kw, mask, rho, u, p = _setup(kind, nx, ny)
    f = _sim(kind, nx, ny, "f64", 0).step(13).populations().cpu().numpy()
    okw = {k: v for k, v in kw.items() if k != "ma"}
    g = O.Grid(9, nx, ny, 1, u_in=(kw.get("ma", 0.0) / np.sqrt(3), 0, 0), mask=mask, **okw)
    g.init(rho, u, p).step(13)
    live = np.ones(nx * ny, bool) if mask is None else mask != W.SOLID
    assert np.abs(f - g.f)[:, live].max() <= F64_TOL * np.abs(g.f).max()


@pytest.mark.parametrize("storage", ["f32", "f16s", "f64"])
@pytest.mark.parametrize("noalloc", [False, True])
def test_batches_of_uneven_steps_equal_single_steps(storage, noalloc):
    """Groups of both paths whose jobs take different numbers of fused and
    single steps, a grid too narrow to be fused among them."""
    import torch
    from paper_1710_02065_amd import lbm
    jobs = [("box", 70, 37, 9), ("box", 3, 40, 6), ("box", 130, 65, 67), ("channel", 200, 90, 3),
            ("noise", 131, 67, 66), ("posts", 129, 23, 0), ("slip", 67, 18, 4)]
    a = [_sim(k, nx, ny, storage, 0) for k, nx, ny, _ in jobs]
    b = [_sim(k, nx, ny, storage, 0) for k, nx, ny, _ in jobs]
    step = lbm.lbm_step_batch_noalloc if noalloc else lbm.lbm_step_batch
    for shift in (0, 1):  # the second call starts from odd times and buffers
        steps = [j[3] + shift for j in jobs]
        step([s.ctx for s in a], steps)
        for s, n in zip(b, steps):
            for _ in range(n):
                s.step(1)
        for s, t, j in zip(a, b, jobs):
            assert s.time == t.time
            assert torch.equal(s.populations(), t.populations()), j


def test_exchange_between_more_slabs_than_one_launch_moves():
    import torch
    from paper_1710_02065_amd import lbm
    from paper_1710_02065_amd.slabs import Slabs
    shape = (33, 45, 1)
    rho, u, p = W.random_state(shape, seed=4, d=2)
    whole = lbm.Simulation(lattice=9, shape=shape, storage="f16s", tau=0.55).init(rho, u, p)
    sl = Slabs(9, shape, lattice=9, storage="f16s", tau=0.55).init(rho, u, p)
    whole.step(6)
    sl.step(6)
    assert torch.equal(whole.populations(), sl.populations())

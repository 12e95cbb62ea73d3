"""Every form of the several-step passes that lbm_step and the batches choose,
against single steps (bitwise) and the oracle (FP64 bar); each case asserts that
the pass is taken.  Completes the sizes of the tests of two and of several
steps: D3Q27 in FP64, whose kernel keeps one plane of each population in LDS, the
64 x 8 tiles with four steps on both paths, and batches with tiles inside the
grid."""
import numpy as np
import pytest

import oracle as O
from tests import test_gpu_several_steps_2d as S2
from tests import test_gpu_two_steps as S3

pytestmark = pytest.mark.gpu

CASES_3D = [(27, (125, 47, 77), "f64", 0), (27, (190, 31, 77), "f64", 1),
            (27, (255, 15, 121), "f64", 0), (27, (250, 131, 97), "f32", 1),
            (27, (256, 128, 128), "f16s", 1), (19, (127, 63, 31), "f64", 0)]


def _equal(a, b, counts):
    import torch
    for n in counts:
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert a.time == b.time
        assert torch.equal(a.populations(), b.populations()), n
    a.sync()


@pytest.mark.parametrize("q,shape,storage,full", CASES_3D)
def test_pairs_equal_single_steps_bitwise(q, shape, storage, full):
    a, b = S3._sim(q, shape, storage, full)[0], S3._sim(q, shape, storage, full)[0]
    assert a.steps_per_pass == 2
    _equal(a, b, (2, 3, 65))


@pytest.mark.parametrize("q,shape,full", [(27, (125, 47, 77), 0), (27, (190, 31, 77), 1),
                                          (19, (127, 63, 31), 0)])
def test_pairs_match_the_oracle_f64(q, shape, full):
    sim, (rho, u, p) = S3._sim(q, shape, "f64", full)
    assert sim.steps_per_pass == 2
    f = sim.step(4).populations().cpu().numpy()
    g = O.Grid(q, *shape, tau=0.53, rho0=1.0625, full_order=bool(full)).init(rho, u, p).step(4)
    assert np.abs(f - g.f).max() <= 1e-12 * np.abs(g.f).max()


# kind, sizes, storages, steps per pass; at 256 compute units grids of 256
# (FP64: 128) tiles and more, of 1024 (256) with walls, take the large tiles
CASES_2D = [("box", 1030, 517, ("f64", "f32", "f32s", "f16s"), 4),
            ("channel", 1001, 701, ("f64", "f32", "f32s"), 4),
            ("noise", 1500, 1333, ("f16s",), 4), ("slip", 1003, 709, ("f64", "f32"), 4),
            ("noise", 1133, 1001, ("f64", "f32", "f32s"), 2),
            ("closed", 300, 201, ("f32", "f16s"), 4), ("posts", 517, 131, ("f32",), 4)]


@pytest.mark.parametrize("kind,nx,ny,storage,steps",
                         [(k, nx, ny, s, n) for k, nx, ny, st, n in CASES_2D for s in st])
@pytest.mark.parametrize("full", [0, 1])
def test_2d_passes_equal_single_steps_bitwise(kind, nx, ny, storage, steps, full):
    a, b = S2._sim(kind, nx, ny, storage, full), S2._sim(kind, nx, ny, storage, full)
    assert a.steps_per_pass == steps
    _equal(a, b, (2, 3, 4, 7, 66))


@pytest.mark.parametrize("kind,nx,ny", [("box", 1030, 517), ("channel", 1001, 701)])
def test_2d_passes_match_the_oracle_f64(kind, nx, ny):
    kw, mask, rho, u, p = S2._setup(kind, nx, ny)
    sim = S2._sim(kind, nx, ny, "f64", 0)
    assert sim.steps_per_pass == 4
    f = sim.step(7).populations().cpu().numpy()
    okw = {k: v for k, v in kw.items() if k != "ma"}
    g = O.Grid(9, nx, ny, 1, u_in=(kw.get("ma", 0.0) / np.sqrt(3), 0, 0), mask=mask, **okw)
    g.init(rho, u, p).step(7)
    live = np.ones(nx * ny, bool) if mask is None else mask != S2.W.SOLID
    assert np.abs(f - g.f)[:, live].max() <= 1e-12 * np.abs(g.f).max()


@pytest.mark.parametrize("storage", ["f32", "f16s", "f64"])
@pytest.mark.parametrize("noalloc", [False, True])
def test_batches_of_wide_grids_equal_single_steps(storage, noalloc):
    """Periodic and walled jobs wide enough for tiles inside the grid, and one too
    narrow to take passes; uneven step counts, from even and odd times."""
    import torch
    from paper_1710_02065_amd import lbm
    jobs = [("box", 260, 141, 9), ("box", 16, 4000, 37), ("box", 513, 65, 67),
            ("channel", 300, 280, 66), ("noise", 331, 267, 35), ("posts", 329, 203, 64),
            ("slip", 367, 318, 5), ("closed", 400, 300, 33), ("channel", 600, 500, 64),
            ("channel", 8, 3000, 21)]
    a = [S2._sim(k, nx, ny, storage, 0) for k, nx, ny, _ in jobs]
    b = [S2._sim(k, nx, ny, storage, 0) for k, nx, ny, _ in jobs]
    step = lbm.lbm_step_batch_noalloc if noalloc else lbm.lbm_step_batch
    for shift in (0, 1):
        steps = [j[3] + shift for j in jobs]
        step([s.ctx for s in a], steps)
        for s, n in zip(b, steps):
            for _ in range(n):
                s.step(1)
        for s, t, j in zip(a, b, jobs):
            assert s.time == t.time
            assert torch.equal(s.populations(), t.populations()), j


@pytest.mark.parametrize("storage", ["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("full", [0, 1])
def test_batched_walls_of_d3q27_equal_the_solo_sweep(storage, full):
    """The batched D3Q27 sweep reads the mask bytes of a wall one by one, the solo
    sweep together: SOLID cells on faces, edges and corners, free-slip and open
    faces beside them."""
    import torch
    from paper_1710_02065_amd import lbm
    sims = []
    for shape, faces in (((21, 14, 11), (2, 2, 1, 1, 2, 2)), ((64, 9, 7), (0, 0, 1, 1, 0, 0))):
        rho, u, p = S2.W.random_state(shape, seed=9, d=3)
        mask = (np.random.default_rng(3).random(rho.size) < 0.15).astype(np.uint8) * S2.W.SOLID
        mask[[0, shape[0] - 1, rho.size - 1]] = S2.W.SOLID
        for _ in range(2):
            sims.append(lbm.Simulation(lattice=27, shape=shape, storage=storage, tau=0.6,
                                       face_bc=faces, flags=lbm.LBM_FULL_ORDER if full else 0)
                        .init(1 + 0.1 * (rho - 1), 0.1 * u, p, mask))
    lbm.lbm_step_batch([s.ctx for s in sims[::2]], [7, 18])
    for s, n in zip(sims[1::2], (7, 18)):
        s.step(n)
    for a, b in zip(sims[::2], sims[1::2]):
        assert torch.equal(a.populations(), b.populations())

"""The choice between passes of several steps and one-step sweeps, evaluated
without a GPU."""
import ctypes as C
import random
import time

import pytest

from paper_1710_02065_amd import lbm

F64, F32, F16S = lbm.LBM_F64, lbm.LBM_F32, lbm.LBM_F16S


def planes(q, storage, nx, ny, nz, cus=256):
    """hrlbm::pair3d_planes: planes per workgroup, 0 for one-step sweeps."""
    fn = lbm.lib()._ZN5hrlbm13pair3d_planesEiijjjj
    fn.argtypes = [C.c_int, C.c_int] + 4 * [C.c_uint32]
    fn.restype = C.c_uint32
    return fn(q, storage, nx, ny, nz, cus)


def iterations(storage, nx, ny, nz, zc, cus=256):
    """Iterations of the busiest compute unit with chunks of zc planes."""
    slots = 2 * cus if storage == F16S else cus
    groups = -(-nx // 64) * -(-ny // 8) * -(-nz // zc)
    return -(-groups // slots) * (zc + 2)


@pytest.mark.parametrize("storage", [F64, F32, F16S])
def test_chunk_length_is_the_best_of_all(storage):
    rng = random.Random(storage)
    taken = 0
    for _ in range(600):
        nx, ny, nz = (int(2 ** rng.uniform(lo, 9.5)) for lo in (5.0, 3.0, 0.0))
        cus = rng.choice([32, 255, 256, 304])
        zc = planes(19, storage, nx, ny, nz, cus)
        if zc:
            taken += 1
            best = min(iterations(storage, nx, ny, nz, -(-nz // c), cus) for c in range(1, nz + 1))
            assert iterations(storage, nx, ny, nz, zc, cus) == best, (nx, ny, nz, cus)
    assert taken > 50  # (the drawn grids reach the pass)


@pytest.mark.parametrize("nx,ny,nz", [(4, 4, 1 << 26), (1, 1, (1 << 31) - 1), (64, 1, 1 << 24),
                                      (1100, 900, 997), (1 << 15, 1 << 15, 1)])
def test_choice_takes_no_time(nx, ny, nz):
    t = time.perf_counter()
    planes(19, F16S, nx, ny, nz)
    assert time.perf_counter() - t < 0.02


def steps2d(general, storage, nx, ny, cus=256):
    """hrlbm::multi2d_steps: steps per pass of a D2Q9 grid, 1 for one-step sweeps."""
    fn = lbm.lib()._ZN5hrlbm13multi2d_stepsEibjjj
    fn.argtypes = [C.c_int, C.c_bool] + 3 * [C.c_uint32]
    return fn(storage, general, nx, ny, cus)


# grids whose pass was measured slower than single steps: lanes of the tiles
# idle, or every tile holds an edge of the grid
NARROW = [(False, F32, 4, 50000), (False, F32, 8, 112500), (False, F16S, 16, 250000),
          (False, F64, 8, 3750), (False, F64, 12, 75000), (True, F32, 8, 25000),
          (True, F32, 32, 28125), (True, F32, 80, 50000), (True, F32, 100000, 9),
          (True, F16S, 40, 100000), (True, F16S, 130, 30769), (True, F16S, 444444, 9),
          (True, F64, 64, 3125), (True, F64, 96, 41666), (True, F64, 197, 561),
          (True, F64, 332, 332), (False, F16S, 3, 5000), (True, F32, 700, 3)]
WIDE = [(False, F32, 4000, 3001, 4), (False, F64, 128, 128, 4), (False, F16S, 12, 60, 4),
        (False, F64, 2048, 1024, 4), (True, F32, 2048, 1024, 2), (True, F64, 2048, 1024, 2),
        (True, F16S, 2048, 1024, 4), (True, F32, 300, 200, 4), (True, F32, 1000, 700, 4)]


@pytest.mark.parametrize("general,storage,nx,ny", NARROW)
def test_narrow_2d_grids_take_single_steps(general, storage, nx, ny):
    assert steps2d(general, storage, nx, ny) == 1


@pytest.mark.parametrize("general,storage,nx,ny,steps", WIDE)
def test_wide_2d_grids_take_passes(general, storage, nx, ny, steps):
    assert steps2d(general, storage, nx, ny) == steps


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("storage,cells", [(F64, 1 << 29), (F32, 1 << 30), (F16S, 1 << 31)])
def test_threads_of_a_2d_pass_fit_a_launch(general, storage, cells):
    """A launch holds less than 2^32 threads; the largest workgroups have 512 for
    64 x 8 cells, so a grid may fill half of them."""
    for nx in list(range(4, 600)) + [2 ** k for k in range(10, 30)]:
        for a, b in ((nx, cells // nx - 1), (cells // nx - 1, nx)):
            if steps2d(general, storage, a, b) > 1:
                assert -(-a // 64) * -(-b // 8) * 512 < 1 << 32, (a, b)

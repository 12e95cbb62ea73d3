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

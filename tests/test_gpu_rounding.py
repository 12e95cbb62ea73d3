"""Rounding of the storages below FP64: the error of a run against the same run
in FP64 (which matches the oracle to 1e-12) may not exceed what is recorded
here."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

STEPS = 60
# density error (over the norm of its fluctuation) and velocity error after
# STEPS steps of the fields below, FP32 storage, of kernels that form a
# population as w (rho0 + drho + ...), per lattice and order: every sum is
# rounded at the size of rho0 there
FP32_BARS = {(9, 0): (1.514e-5, 1.683e-6), (9, 1): (1.631e-5, 1.773e-6),
             (19, 0): (3.655e-5, 1.450e-6), (27, 0): (3.632e-5, 1.242e-6),
             (27, 1): (4.072e-5, 1.538e-6)}


def _fields(shape):
    """Taylor-Green vortex with a density pulse."""
    nx, ny, nz = shape
    c = np.arange(nx * ny * nz)
    x, y, z = c % nx, (c // nx) % ny, c // (nx * ny)
    px, py, pz = 2 * np.pi * x / nx + 1, 2 * np.pi * y / ny + 2, 2 * np.pi * z / nz + 0.5
    cz = np.cos(pz) if nz > 1 else 1.0
    U = 0.1 / np.sqrt(3)
    u = np.zeros((3, c.size))
    u[0], u[1] = U * np.sin(px) * np.cos(py) * cz, -U * np.cos(px) * np.sin(py) * cz
    rho = 1 + 3 * U * U / 16 * (np.cos(2 * px) + np.cos(2 * py)) * (cz * cz + 1)
    d2 = (x - nx / 3) ** 2 + (y - ny / 2) ** 2 + (z - nz / 2) ** 2
    return rho + 1e-3 * np.exp(-d2 / 30), u


def errors(q, full, storage):
    """(density error, velocity error) of STEPS steps against FP64."""
    from paper_1710_02065_amd import lbm
    shape = (160, 130, 1) if q == 9 else (48, 44, 40)
    rho, u = _fields(shape)
    out = []
    for st in ("f64", storage):
        sim = lbm.Simulation(lattice=q, shape=shape, storage=st, tau=0.52,
                             flags=lbm.LBM_FULL_ORDER if full else 0)
        out.append([v.double().cpu().numpy() for v in sim.init(rho, u).step(STEPS).moments()])
        sim.close()
    (r0, u0), (r1, u1) = out
    norm = np.linalg.norm
    return norm(r1 - r0) / norm(r0 - r0.mean()), norm(u1 - u0) / norm(u0)


@pytest.mark.parametrize("q,full", sorted(FP32_BARS))
def test_fp32_error_stays_below_the_recorded_one(q, full):
    e_rho, e_u = errors(q, full, "f32")
    assert e_rho <= FP32_BARS[q, full][0] and e_u <= FP32_BARS[q, full][1], (e_rho, e_u)


@pytest.mark.parametrize("width", [3, 49, 103, 197, 321])
def test_fp32_layer_strength_is_of_the_correctly_rounded_distance(width):
    """One step from rest with a moving reference state: the momentum of a cell
    in the layer gives its strength chi.  With d = (s - s0) / W rounded once,
    the rest of chi and the collision is about 30 roundings; d a rounding
    further off changes 1 - d, and with it chi, by W roundings in the
    outermost cells.  (Storage of deviations: a population that carries its
    rest part has no digits for the small momenta.)"""
    from paper_1710_02065_amd import lbm
    nx, U, chi_max = width + 7, 0.1, 0.2
    sim = lbm.Simulation(lattice=9, shape=(nx, 6, 1), storage="f32s", tau=0.6,
                         face_bc=(2, 2, 0, 0, 0, 0), sponge_width=(0, width, 0, 0, 0, 0),
                         chi_max=chi_max, rho_ref=1.0, u_ref=(U, 0.0, 0.0))
    f = sim.init().step(1).populations().cpu().numpy().reshape(9, 6, nx)
    xi, _ = lbm.lbm_lattice_table(9)
    j = np.tensordot(xi[:, 0].astype(float), f, 1)[3]
    s = np.arange(nx) - (nx - width)
    d = np.maximum(s.astype(np.float32) / np.float32(width), 0).astype(np.float64)
    chi = chi_max * 3125 / 256 * (1 - d) * d ** 4
    want = (1 - chi) * 0.5 * chi * U / (1 + 0.5 * chi) + chi * U
    inside = want > 0
    assert inside.sum() == width - 1
    assert np.abs(j[inside] / want[inside] - 1).max() <= 32 * 2.0 ** -24
    assert np.abs(j[~inside]).max() <= 1e-13

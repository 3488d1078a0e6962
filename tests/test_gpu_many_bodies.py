"""GPU: the phase update for more than four bodies (its variants for up to 8 and up to 16) against the FP64
oracle at round-off, on a ragged grid with interface energies that differ from pair to pair.

The update takes the bodies active on a tile: one, two, three or four of them (the others zero there), or
all of them when five or more are active.  The placement puts every one of these lists on some tile, which the test
checks by counting, per 8 x 8 x 4 tile, the bodies whose interface lies on it or a neighbour."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from parity_helpers import compare, log  # noqa: E402
from pflbm_inputs import coexistence_densities, default_params, liquid_density, sphere_phi  # noqa: E402
from pflbm_inputs.geometry import grid, mimg  # noqa: E402

FP64 = dict(tol_field=1e-11, tol_force=1e-9, tol_node=1e-10)
SHAPE = (22, 37, 83)


def many_bodies(nb):
    """nb spheres, x positions thinning out along the box, in and around a drop."""
    from pflbm_inputs.workloads import Workload
    nz, ny, nx = SHAPE
    rng = np.random.default_rng(100 + nb)
    phis, bodies = [], []
    for a in range(nb):
        c = (8.0 + 62.0 * ((a + 0.5) / nb) ** 2.5, 8.0 + 20.0 * rng.random(), 5.0 + 12.0 * rng.random())
        phis.append(sphere_phi(SHAPE, c, 3.2 + 0.8 * rng.random(), 2.5))
        bodies.append(dict(mass_density=3.0, wetting_rho=0.8 + 0.04 * a, v=list(0.02 * rng.standard_normal(3)),
                           w=list(0.005 * rng.standard_normal(3)), fixed=0))
    phi = np.stack(phis)
    s = phi.sum(0)
    phi = np.where(s > 1, phi / np.where(s > 1, s, 1), phi)
    rv, rl = coexistence_densities()
    x, y, z = grid(SHAPE)
    d = np.sqrt(mimg(x - 20, nx) ** 2 + mimg(y - 18, ny) ** 2 + mimg(z - 11, nz) ** 2) - 9.0
    sigma = rng.uniform(0.4, 1.2, (nb + 1, nb + 1))
    sigma = 0.5 * (sigma + sigma.T)
    np.fill_diagonal(sigma, 0.0)
    return Workload("many bodies", default_params(nx, ny, nz, nb, e0=0.5, mobility=1e-3, sigma=sigma), bodies,
                    liquid_density(d, rl, rv, 3.0), phi)


def active_counts(phi):
    """Bodies with an interface on a tile or one of its 26 neighbours, for every tile."""
    nb = phi.shape[0]
    tiles = [-(-n // t) for n, t in zip(SHAPE, (4, 8, 8))]
    mixed = np.zeros([nb] + tiles, dtype=bool)
    for k in np.ndindex(*tiles):
        b = phi[:, 4 * k[0]:4 * k[0] + 4, 8 * k[1]:8 * k[1] + 8, 8 * k[2]:8 * k[2] + 8].reshape(nb, -1)
        mixed[(slice(None),) + k] = (b != 0).any(1) & (b != 1).any(1)
    act = np.zeros_like(mixed)
    for d in np.ndindex(3, 3, 3):
        act |= np.roll(mixed, [v - 1 for v in d], axis=(1, 2, 3))
    return act.sum(0)


@pytest.mark.parametrize("nb", [5, 8, 9, 16])
def test_many_bodies_fp64(oracle_mod, nb):
    from paper_1902_10432_amd.simulation import Simulation
    steps = 20
    w = many_bodies(nb)
    counts = np.bincount(active_counts(w.phi0).reshape(-1), minlength=nb + 1)
    log(f"case {nb} bodies, tiles by active bodies {counts.tolist()}")
    assert all(counts[k] > 0 for k in range(1, 5)) and (nb == 5 or counts[5:].sum() > 0)
    sim = Simulation(w.params, w.bodies, w.rho0, w.phi0, precision="fp64")
    sim.step(steps)
    ref = oracle_mod.Oracle(w.params, w.bodies, w.rho0, w.phi0)
    ref.step(steps)
    compare(sim, ref, steps, lever=3.0, **FP64)
    vol_g, vol_o = sim.phi().sum((1, 2, 3)), ref.phi().sum((1, 2, 3))
    assert np.abs(vol_g - vol_o).max() <= 1e-10 * vol_o.max()
    assert sim.diag()["n_f2s"] == ref.diag()["n_f2s"] and sim.diag()["n_s2f"] == ref.diag()["n_s2f"]
    assert (sim.mask()[1].max() + 1) == nb  # every body holds solid nodes

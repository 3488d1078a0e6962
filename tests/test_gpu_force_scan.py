"""GPU: the force scan's repulsion search and link sums against the FP64 oracle where its branches
can go wrong: three spheres that nearly touch (a solid node meets several bodies within r_c), search
radii from no offset at all to the largest (r_c = 4: 250 offsets, four rounds of 64 lanes), axes
shorter than twice the reach, and every sphere moving and rotating.

Both sides compute in FP64 from the same inputs and differ by summation order only: a force is a sum
of about 10^3 terms of order one that cancels to order 0.1, so 10^3 * 2^-53 / 0.1 ~ 1e-12 relative to
the largest component; the bound is 1e-10 after three steps.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from pflbm_inputs import default_params  # noqa: E402
from pflbm_inputs.geometry import sphere_phi  # noqa: E402


@pytest.mark.parametrize("shape,rc,lattice", [((17, 19, 23), 1.0, 19), ((17, 19, 23), 3.0, 19), ((17, 19, 23), 4.0, 19),
                                              ((7, 18, 21), 4.0, 27), ((40, 33, 66), 3.0, 19)])
def test_three_spheres_in_contact_fp64(shape, rc, lattice):
    import oracle
    from paper_1902_10432_amd.simulation import Simulation
    print(f"case {shape} rc={rc} lattice={lattice}", flush=True)
    oracle.build(force=False)
    nz, ny, nx = shape
    r = 4.2 if nz > 8 else 2.6
    mid = np.array([nx, ny, nz]) / 2.0
    centres = [mid + np.array(d) * 1.02 * r for d in ((-1.0, -0.6, 0.1), (1.0, -0.6, -0.1), (0.0, 1.1, 0.05))]
    phi = np.stack([sphere_phi(shape, c, r, 1.5) for c in centres])
    total = phi.sum(0)
    phi = np.where(total > 1.0, phi / np.where(total > 1.0, total, 1.0), phi)
    rng = np.random.default_rng(5)
    rho = 0.4 + 0.05 * rng.random(shape)
    bodies = [{"mass_density": 4.0, "wetting_rho": 1.0 + 0.1 * k, "fixed": 0, "v": tuple(rng.uniform(-0.01, 0.01, 3)),
               "w": tuple(rng.uniform(-0.005, 0.005, 3))} for k in range(3)]
    p = default_params(nx, ny, nz, 3, tau=1.1, rc=rc, e0=0.4, lattice=lattice)
    sim = Simulation(p, bodies, rho, phi, precision="fp64")
    ref = oracle.Oracle(p, bodies, rho, phi)
    sim.step(3)
    ref.step(3)
    got, want = sim.bodies(), ref.bodies()
    for k in ("F", "T"):
        err = np.abs(got[k] - want[k]).max() / np.abs(want[k]).max()
        print(f"  {k}: {err:.2e}", flush=True)
        assert err <= 1e-10
    rel = np.linalg.norm(sim.rho() - ref.rho()) / np.linalg.norm(ref.rho())
    assert rel <= 1e-11

"""GPU: the two forms of the FP32 D3Q27 fluid pass in tiles of 8 rows (two blocks a CU, and one on large grids)
give the bits of the 4-row tile, on both sides of the rule: a small grid, rows that fill their tiles on grids
just below and above 6 million nodes, rows that fill three quarters of theirs just above 9.5 million."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from pflbm_inputs import tiny_moving_body  # noqa: E402


@pytest.mark.parametrize("shape", [(5, 199, 201), (236, 198, 128), (238, 198, 128), (241, 198, 200)])
def test_forms_are_bit_identical(shape):
    from paper_1902_10432_amd.simulation import Simulation
    w = tiny_moving_body(shape=shape, second_body=True, lattice=27, tau=1.1)

    def state(tile):
        print(f"case {shape} tile {tile}", flush=True)
        s = Simulation(w.params, w.bodies, w.rho0, w.phi0, precision="fp32")
        if tile:
            s.set_tile(*tile)
        s.step(5)
        out = [s.rho(), s.phi()] + [s.bodies()[k] for k in ("F", "T", "X", "V", "W")]
        s.close()
        return out

    ref = state((4, 8))
    for tile in (None, (8, 3)):
        for a, b in zip(ref, state(tile)):
            assert np.array_equal(a, b)

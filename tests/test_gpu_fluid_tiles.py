"""GPU: the fluid pass gives the same bits whatever its tile, down to z-chunks of one plane (more
blocks than planes on the axis, chunks that do not divide it), on every precision and lattice: the
tile only splits the work.  The extra block that publishes the step state runs in each."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from pflbm_inputs import tiny_moving_body  # noqa: E402


@pytest.mark.parametrize("lattice", [19, 27])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16"])
def test_tiles_are_bit_identical(precision, lattice):
    from paper_1902_10432_amd.simulation import Simulation
    w = tiny_moving_body(shape=(11, 13, 70), second_body=True, lattice=lattice, tau=1.1)

    def state(tile):
        print(f"case {precision} d3q{lattice} tile {tile}", flush=True)
        s = Simulation(w.params, w.bodies, w.rho0, w.phi0, precision=precision)
        if tile:
            s.set_tile(*tile)
        s.step(6)
        return [s.rho(), s.mom(), s.phi()] + [s.bodies()[k] for k in ("F", "T", "X", "V", "W")]

    ref = state((4, 8))
    for tile in (None, (4, 1), (4, 3), (4, 64)):
        for a, b in zip(ref, state(tile)):
            assert np.array_equal(a, b)

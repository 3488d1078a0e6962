"""GPU: the autotuner times the shape in use beside its own candidates, so that tuning cannot leave a run
slower than it was: with a chunk that is not among the candidates it takes the steps of one more."""
import pytest

pytestmark = pytest.mark.gpu

from pflbm_inputs import bridge_pair  # noqa: E402


@pytest.mark.parametrize("precision,candidates", [("fp32", 6), ("fp64", 3)])
def test_present_shape_is_timed(precision, candidates):
    """16 <= nz < 32: chunks of 4, 8 and 16 planes for each of the rows built (4 and 8, FP64: 4)."""
    from paper_1902_10432_amd.simulation import Simulation
    print(f"case autotune {precision}", flush=True)
    w = bridge_pair((20, 26, 36), 4.5, 5.0, 2.5, 0.10, 10.0)
    for planes, extra in ((8, 0), (5, 1), (1, 1), (20, 1), (32, 1)):
        sim = Simulation(w.params, w.bodies, w.rho0, w.phi0, precision=precision)
        sim.set_tile(4, planes)
        t = sim.autotune(2)
        taken = sim.diag()["step"]
        print(f"  {planes} planes: {t}, {taken} steps", flush=True)
        assert t["tile_rows"] in (4, 8) and t["chunk_planes"] in (4, 8, 16)
        assert taken == 3 * (candidates + extra)
        sim.close()

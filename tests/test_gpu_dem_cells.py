"""GPU: the cell grid of the many-sphere run where the wrap into the box rounds: a sphere that moved more
than 2^53 boxes in a step lands outside [0, L), where its minimum images are still well defined."""
import math
from fractions import Fraction

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import dem_oracle as D  # noqa: E402

NORM = {"in_shift": [0.2, 0.8, 0.5, 0.5], "in_scale": [3.0, 5.0, 2.0, 2.0], "out_shift": 0.5, "out_scale": 0.3}


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_far_sphere_keeps_its_bridges(sign):
    from paper_1902_10432_amd.surrogate import SphereRun, Surrogate, dem_config
    print(f"case far sphere {sign}", flush=True)
    n, gap_max = 2048, 1.5
    rng = np.random.default_rng(2)
    R = rng.uniform(2.0, 3.0, n)
    L = (n * 4.0 / 3.0 * math.pi * 2.5 ** 3 / 0.2) ** (1.0 / 3.0)
    x = rng.uniform(0.0, L, (n, 3))
    # a velocity whose step (dt 1) lands more than two cells outside the box
    v0 = sign * 1.2e19
    while True:
        v0 = float(np.nextafter(v0, sign * np.inf))
        k = math.floor(v0 / L)
        land = float(Fraction(v0) - Fraction(L) * k)
        if (land < -20.0 or land > L + 20.0) and 20.0 < land % L < L - 20.0:
            break
    v = np.zeros((n, 3))
    v[0, 0] = v0
    net = Surrogate(4, 64, 2, max_batch=65536, seed=3)
    cfg = dem_config(n, L, 1.0, 1e12, 4.0, 0.0, 0.5, 0.05, 0.25, gap_max, NORM, max_neighbours=64, max_pairs=65536)
    run = SphereRun(net, cfg, R, x, v)
    run.step(1)
    xs = run.state()["x"]
    print(f"  lands at {xs[0, 0]:.3f} of {L:.3f}", flush=True)
    assert not 0.0 <= xs[0, 0] < L
    run.evaluate()
    ij = D.bridges(xs, R, L, gap_max)[0]
    assert (ij[:, 0] == 0).sum() >= 2
    assert np.array_equal(run.pairs()["ij"], ij)

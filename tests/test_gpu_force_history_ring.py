"""GPU: the force history once its ring of 8192 steps has wrapped: windows that end before, at and
after the wrap, and one whole ring, against the forces recorded earlier; exact (FP64 copies)."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from pflbm_inputs import bridge_pair  # noqa: E402

RING = 8192


def _print(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def test_history_windows_across_the_ring_end():
    import torch
    assert torch.cuda.is_available()
    from paper_1902_10432_amd.simulation import Simulation
    w = bridge_pair((20, 26, 36), 4.5, 5.0, 2.5, 0.10, 10.0)
    _print(f"case force history of {RING + 9} steps, {w.shape}")
    s = Simulation(w.params, w.bodies, w.rho0, w.phi0, precision="fp32")
    s.step(RING - 6)
    before = s.force_history(RING)  # no wrap yet
    assert before.shape == (RING - 6, len(w.bodies), 6)
    late = []
    for _ in range(15):
        s.step(1)
        b = s.bodies()
        late.append(np.concatenate([b["F"], b["T"]], axis=1))
    every = np.concatenate([before, np.stack(late)])
    for n in (0, 1, 8, 9, 10, 15, 300, RING, RING + 5):
        h = s.force_history(n)
        assert np.array_equal(h, every[len(every) - min(n, RING):]), n

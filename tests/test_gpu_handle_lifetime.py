"""GPU: a handle or a batch released after its streams, as it may be once its results have been read: the
release waits for captured steps that may still run, and touches no stream of the caller's then."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from pflbm_inputs import bridge_pair  # noqa: E402

PAIR = ((24, 28, 40), 5.0, 6.5, 3.0, 0.05, 30.0)


def _stream(lib):
    import torch
    s = C.c_void_p()
    assert lib.hipStreamCreate(C.byref(s)) == 0
    return s, torch.cuda.ExternalStream(s.value)


@pytest.mark.parametrize("steps", [1, 2, 35])
def test_handle_after_its_stream(steps):
    import torch
    from paper_1902_10432_amd import binding as B
    from paper_1902_10432_amd.simulation import Simulation
    print(f"case handle after its stream, {steps} steps", flush=True)
    torch.cuda.init()
    lib, w = B.load_library(), bridge_pair(*PAIR)
    s, ext = _stream(lib)
    sim = Simulation(w.params, w.bodies, w.rho0, w.phi0, precision="fp32", stream=ext)
    ref = Simulation(w.params, w.bodies, w.rho0, w.phi0, precision="fp32")
    sim.step(steps)
    ref.step(steps)
    F = sim.bodies()["F"]
    assert np.array_equal(F, ref.bodies()["F"])
    assert lib.hipStreamDestroy(s) == 0
    sim.close()
    ref.step(2)      # queued steps on a live stream: the release waits for them
    ref.close()


def test_batch_after_its_streams():
    import torch
    from paper_1902_10432_amd import binding as B
    from paper_1902_10432_amd.simulation import Batch, Simulation
    print("case batch after its streams", flush=True)
    torch.cuda.init()
    lib, w = B.load_library(), bridge_pair(*PAIR)
    streams = [_stream(lib) for _ in range(2)]
    sims = [Simulation(w.params, w.bodies, w.rho0, w.phi0, precision="fp32", stream=e) for _, e in streams]
    b = Batch(sims, graph_steps=2)
    b.step(6)
    F = [s.bodies()["F"] for s in sims]
    assert np.array_equal(F[0], F[1])
    for s in sims:
        s.close()
    for s, _ in streams:
        assert lib.hipStreamDestroy(s) == 0
    b.close()

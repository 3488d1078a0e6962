"""GPU: what the many-sphere run does when a call is refused or fails: the state and the bridge list stay
those of the last evaluation that succeeded."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NORM = {"in_shift": [0.2, 0.8, 0.5, 0.5], "in_scale": [3.0, 5.0, 2.0, 2.0], "out_shift": 0.5, "out_scale": 0.3}
THETA, CFRAC = 0.5, 0.05


def _run(L, R, x, v, cap=16, max_pairs=256, hidden=64):
    from paper_1902_10432_amd.surrogate import SphereRun, Surrogate, dem_config
    net = Surrogate(4, hidden, 2, max_batch=max(256, max_pairs), seed=3)
    cfg = dem_config(len(R), L, 1.0, 1e6, 4.0, 0.5, THETA, CFRAC, 0.25, 1.5, NORM, max_neighbours=cap,
                     max_pairs=max_pairs)
    return SphereRun(net, cfg, R, x, v)


def _state(run):
    s = run.state()
    return [s[k] for k in ("x", "v", "F")]


@pytest.mark.parametrize("hidden", [64, 48])
def test_captured_stream_is_refused(hidden):
    """A run on a stream that is being captured is refused (it waits for the stream); the state and the
    run that follows are those of a run that never tried, after an odd number of steps too."""
    from paper_1902_10432_amd import binding as B
    from paper_1902_10432_amd.surrogate import SurrogateError
    print(f"case captured stream hidden={hidden}", flush=True)
    rng = np.random.default_rng(5)
    L, R = 40.0, rng.uniform(2.0, 3.0, 60)
    x, v = rng.uniform(0.0, L, (60, 3)), rng.normal(0.0, 0.05, (60, 3))
    run, ref = _run(L, R, x, v, 32, hidden=hidden), _run(L, R, x, v, 32, hidden=hidden)
    run.step(2)
    ref.step(2)
    lib, stream = B.load_library(), C.c_void_p(run.net.stream.cuda_stream)
    for call in (lambda: run.step(1), run.evaluate, lambda: run.step(3)):
        graph = C.c_void_p()
        assert lib.hipStreamBeginCapture(stream, 2) == 0  # relaxed: other streams and threads go on
        with pytest.raises(SurrogateError):
            call()
        rc = lib.hipStreamEndCapture(stream, C.byref(graph))
        if graph.value:
            lib.hipGraphDestroy(graph)
        print(f"  end of capture: {rc}", flush=True)
        for a, b in zip(_state(run), _state(ref)):
            assert np.array_equal(a, b)
    run.step(2)
    ref.step(2)
    for a, b in zip(_state(run), _state(ref)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("cap,max_pairs,match", [(1, 256, "max_neighbours"), (8, 3, "max_pairs")])
def test_overflow_keeps_the_bridge_list(cap, max_pairs, match):
    """A sphere of the lowest index flies at one of three bridged pairs: the evaluation that finds the
    fourth bridge, ahead of the others in the list, overflows.  Pairs, features and forces are then
    those of the evaluation before it, also when the run goes on for an even or odd number of steps."""
    from paper_1902_10432_amd.surrogate import SurrogateError
    print(f"case overflow cap={cap} max_pairs={max_pairs}", flush=True)
    L, R = 80.0, np.array([2.0, 2.1, 2.2, 2.3, 2.4, 2.5, 2.6])
    x = np.array([[20.0, 31.0, 20.0], [20.0, 20.0, 20.0], [25.0, 20.0, 20.0], [50.0, 20.0, 20.0], [55.2, 20.0, 20.0],
                  [50.0, 60.0, 20.0], [50.0, 65.8, 20.0]])
    v = np.zeros((7, 3))
    v[0, 1], v[1, 0], v[3, 0], v[5, 1] = -1.0, 0.003, -0.004, 0.005  # the features change every step
    ref, good = _run(L, R, x, v, 8), 0
    while True:  # steps until the evaluation at the reached positions finds the fourth bridge
        ref.evaluate()
        if len(ref.pairs()["ij"]) > 3:
            break
        ref.step(1)
        good += 1
    assert 2 <= good < 20
    ref = _run(L, R, x, v, 8)
    ref.step(good)
    want, state = ref.pairs(), _state(ref)
    assert len(want["ij"]) == 3
    for extra in (1, 2, 5):
        run = _run(L, R, x, v, cap, max_pairs)
        with pytest.raises(SurrogateError, match=match):
            run.step(good + extra)
        for a, b in zip(_state(run), state):
            assert np.array_equal(a, b)
        for _ in range(2):
            got = run.pairs()
            for k in ("ij", "features", "force"):
                assert np.array_equal(got[k], want[k]), k
            with pytest.raises(SurrogateError, match=match):
                run.evaluate()

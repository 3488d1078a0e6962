"""GPU: the network's output written into the memory of its inputs (a program that no longer needs them).
The one-launch pass reads inputs and writes outputs in one kernel, so such a call has to take the path that
copies the inputs first.  Same products either way, output sums in another order: 1e-5 of the RMS, as
between the two passes in test_gpu_mlp.py."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,n,at", [(256, 65536, 3 * 65536), (128, 65536, 3 * 65536), (64, 65536, 3 * 65536),
                                         (256, 65536, 0), (48, 4097, 0), (128, 700, 4 * 700 - 1), (128, 700, 4 * 700)])
def test_output_over_the_inputs(hidden, n, at):
    """at: where the outputs begin, in floats from the inputs (the last case only touches them)."""
    import torch
    from paper_1902_10432_amd import binding as B
    from paper_1902_10432_amd.surrogate import Surrogate
    print(f"case hidden={hidden} n={n} at={at}", flush=True)
    net = Surrogate(4, hidden, 3, max_batch=n, seed=hidden)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    x = torch.randn((n, 4), generator=gen, device="cuda", dtype=torch.float32)
    want = net.forward(x).cpu().numpy()
    buf = torch.empty(5 * n, device="cuda", dtype=torch.float32)
    buf[:4 * n] = x.reshape(-1)
    torch.cuda.synchronize()
    rc = B.load_library().pf_mlp_forward(net._h, C.c_void_p(buf.data_ptr()), n, C.c_void_p(buf.data_ptr() + 4 * at))
    assert rc == 0
    net.stream.synchronize()
    got = buf[at:at + n].cpu().numpy()
    rms = float(np.sqrt((want.astype(np.float64) ** 2).mean()))
    err = float(np.abs(got - want).max()) / rms
    print(f"  max difference {err:.2e} of the RMS", flush=True)
    assert err <= 1e-5

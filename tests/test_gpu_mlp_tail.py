"""GPU: SiLU and its derivative where the sigmoid's denominator 1 + exp(-z) nears the largest FP32 value (z
from -80 to -88.7), in the fused passes (widths 64, 256) and layer by layer (48).

One hidden unit has pre-activation z (its bias) and output weight 2^118, so the output is
bf16(silu(z)) 2^118.  Bound: one BF16 step (2^-8) for the activation, which the relative error of FP32
exp(-z) (its argument in FP32, 2^-18) moves at most to the next step.  The bias gradient 2 y 2^118
silu'(z) passes the BF16 output gradient and FP32: two BF16 steps (2^-7)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import mlp_oracle as M  # noqa: E402


@pytest.mark.parametrize("hidden", [48, 64, 256])
@pytest.mark.parametrize("z", [-80.0, -87.0, -87.5, -88.0, -88.7])
def test_silu_tail(hidden, z):
    import torch
    from paper_1902_10432_amd.surrogate import Surrogate
    print(f"case hidden={hidden} z={z}", flush=True)
    net = Surrogate(1, hidden, 1, max_batch=64, seed=0)
    p = np.zeros(net.n_params, dtype=np.float32)
    p[hidden + 3] = z                      # bias of unit 3
    p[2 * hidden + 3] = 2.0 ** 118         # its output weight
    net.set_params(p)
    x = torch.zeros((1, 1), dtype=torch.float32, device="cuda")
    zf = np.float64(np.float32(z))
    want = M.silu(zf) * 2.0 ** 118
    y = float(net.forward(x)[0])
    assert abs(y - want) <= 2.0 ** -8 * abs(want), (y, want)
    _, g = net.gradients(x, torch.zeros(1, dtype=torch.float32, device="cuda"))
    gw = 2.0 * want * 2.0 ** 118 * M.silu_grad(zf)
    assert abs(float(g[hidden + 3]) - gw) <= 2.0 ** -7 * abs(gw), (g[hidden + 3], gw)

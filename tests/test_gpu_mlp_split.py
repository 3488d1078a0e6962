"""GPU: gradients where the split of the batch or the width of the network picks another path, against
the FP64 network oracle with BF16 operand rounding: widths with a one-launch pass (64, 128, 256) and
without one (48, 160: two column tiles of the weight gradient), one row, the edges of the 16-row
blocks and 32-row chunk steps, the last batch of 16-row blocks and the first of 64-row blocks, one
and eight hidden layers, three inputs (element loads).

Bounds as in test_gpu_mlp.py: the kernels differ from that oracle by FP32 accumulation order and the
BF16 rounding of the back-propagated error, 2^-9 through up to nine products: 1.5e-2 relative per layer,
2e-3 for the loss.  With eight layers a rounding can move an activation by one BF16 step that the next
layers carry on, so the bound doubles.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import mlp_oracle as M  # noqa: E402


@pytest.mark.parametrize("n_in,hidden,layers,n", [
    (4, 128, 1, 1), (3, 64, 2, 15), (4, 256, 2, 17), (4, 128, 8, 33), (4, 160, 2, 65), (4, 48, 3, 97),
    (4, 64, 2, 8192), (4, 64, 2, 8193), (16, 128, 3, 3105),
])
def test_gradients_over_splits(n_in, hidden, layers, n):
    import torch
    from paper_1902_10432_amd.surrogate import Surrogate
    print(f"case n_in={n_in} hidden={hidden} layers={layers} n={n}", flush=True)
    net = Surrogate(n_in, hidden, layers, max_batch=max(n, 64), seed=n)
    rng = np.random.default_rng(n)
    p = M.to_bf16(net.params()).astype(np.float32)
    k = 0
    for o, i in M.layer_shapes(n_in, hidden, layers):
        k += o * i
        p[k:k + o] = rng.normal(0.0, 0.2, o).astype(np.float32)
        k += o
    net.set_params(p)
    x = rng.normal(0.0, 1.0, (n, n_in)).astype(np.float32)
    t = rng.normal(0.0, 1.0, n).astype(np.float32)
    loss, g = net.gradients(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda())
    lb, gb = M.loss_and_grad(p.astype(np.float64), x, t, n_in, hidden, layers, bf16_acts=True)
    scale = 2.0 if layers == 8 else 1.0
    assert abs(loss - lb) <= scale * 2e-3 * lb
    k = 0
    for layer, (o, i) in enumerate(M.layer_shapes(n_in, hidden, layers)):
        for name, size in (("W", o * i), ("b", o)):
            a, b = g[k:k + size], gb[k:k + size]
            err = float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))
            print(f"  layer {layer} {name}: {err:.2e}", flush=True)
            assert err <= scale * 1.5e-2, (layer, name)
            k += size

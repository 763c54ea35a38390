"""The one-kernel training step of the MLP against the FP64 CPU oracle at the edges of
its shapes: one row, rows past a tile and past one tile per compute unit (shares added
to), outputs at and past a chunk of 64, hidden widths at 64, 65 and 128, inputs up to
32, and the first widths that the layer-by-layer path still takes (33 inputs, 129
hidden).  FP32 against FP64: losses and gradients within a relative 1e-4, the tolerance
of the layer-by-layer path's test; two runs agree bit for bit."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1706_10086_amd as mg  # noqa: E402
from oracle import mlp as omlp  # noqa: E402


@pytest.mark.parametrize("I,H,O,B", [(1, 1, 1, 1), (6, 64, 64, 64), (6, 64, 65, 65), (32, 64, 128, 257),
                                     (32, 65, 63, 33), (7, 128, 200, 500), (33, 64, 20, 90),
                                     (6, 129, 20, 90), (6, 64, 30, 40001), (5, 100, 10, 20001)])
def test_step_matches_oracle(I, H, O, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"mlp step I={I} H={H} O={O} B={B}", flush=True)
    dev = torch.device("cuda:0")
    seed = I + H + O + B
    theta = omlp.he_uniform_init(I, H, O, seed)
    theta = (theta + 0.05 * synth.uniform_pm1(theta.shape, seed + 5)).astype(np.float32)
    X = synth.uniform_pm1((B, I), seed + 1).astype(np.float32)
    T = (0.5 + 0.5 * synth.uniform_pm1((B, O), seed + 2)).astype(np.float32)
    M = (synth.unit(seed + 3, B * O) < 0.6).astype(np.float32).reshape(B, O)
    M[0, 0] = 1.0
    grads = []
    for _ in range(2):
        net = mg.MLP(I, H, O, theta)
        net.set_data(*(torch.from_numpy(x).to(dev) for x in (X, T, M)))
        loss, g = net.loss_grad()
        grads.append(g)
        # a training step leaves the loss it was taken at
        assert net.train(1) == loss
        net.destroy()
    want_loss, want = omlp.loss_and_grad(theta.astype(np.float64), X, T, M, I, H, O)
    assert abs(loss - want_loss) <= 1e-4 * abs(want_loss)
    assert np.linalg.norm(grads[0] - want) <= 1e-4 * np.linalg.norm(want)
    assert np.array_equal(grads[0], grads[1])

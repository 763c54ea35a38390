"""Networks on both sides of the line between the step kernel and the layer-by-layer
path (few rows against many outputs; rounds of row tiles above 64 hidden units) against
the FP64 CPU oracle.  FP32 against FP64: losses and gradients within a relative 1e-4, the
tolerance of the two paths' own tests."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1706_10086_amd as mg  # noqa: E402
from oracle import mlp as omlp  # noqa: E402


@pytest.mark.parametrize("I,H,O,B", [(6, 64, 769, 768), (6, 64, 769, 769), (6, 128, 1024, 8200),
                                     (6, 128, 1025, 8200), (6, 65, 2049, 300)])
def test_both_paths_match_oracle(I, H, O, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"mlp routes I={I} H={H} O={O} B={B}", flush=True)
    dev = torch.device("cuda:0")
    seed = 3 * I + H + O + B
    theta = omlp.he_uniform_init(I, H, O, seed)
    X = synth.uniform_pm1((B, I), seed + 1).astype(np.float32)
    T = (0.5 + 0.5 * synth.uniform_pm1((B, O), seed + 2)).astype(np.float32)
    M = (synth.unit(seed + 3, B * O) < 0.6).astype(np.float32).reshape(B, O)
    net = mg.MLP(I, H, O, theta)
    net.set_data(*(torch.from_numpy(x).to(dev) for x in (X, T, M)))
    loss, g = net.loss_grad()
    # a training step leaves the loss it was taken at
    assert net.train(1) == loss
    net.destroy()
    want_loss, want = omlp.loss_and_grad(theta.astype(np.float64), X, T, M, I, H, O)
    assert abs(loss - want_loss) <= 1e-4 * abs(want_loss)
    assert np.linalg.norm(g - want) <= 1e-4 * np.linalg.norm(want)

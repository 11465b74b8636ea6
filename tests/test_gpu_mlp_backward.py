"""The MLP's backward kernel at the edges of its tiles: 16 samples a tile, 16
waves of tiles (256 samples) a round; fewer samples than a tile, one more and
one less, a last round with one tile, against the FP64 oracle on the FP32
activations.  Tolerance: products and sums of at most 64 x 3 and 1024 terms in
FP32 (6e-8 each, random signs) and activations 1e-6 off, so 1e-4 of the largest
gradient, as for the forward and backward pass together."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 255, 256, 272, 1024])
def test_backward_at_tile_edges(B):
    import torch
    import paper_2307_12276_amd as A
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(B)
    Wh = mlp.init_params(7).astype(np.float32)
    X = rng.standard_normal((B, 9)).astype(np.float32)
    dYh = rng.standard_normal((B, 3)).astype(np.float32)
    _, co = mlp.forward(Wh.astype(np.float64), X.astype(np.float64))
    go = mlp.backward(Wh.astype(np.float64), co, dYh.astype(np.float64))
    Wd, dY = torch.from_numpy(Wh).to(dev), torch.from_numpy(dYh).to(dev)
    cache = torch.from_numpy(np.concatenate(co, axis=1).astype(np.float32)).to(dev)
    # (rows past the batch must not be read into any sum)
    cache = torch.cat([cache, torch.full((16, cache.shape[1]), float("nan"), device=dev)])[:B]
    out = []
    for _ in range(2):
        dW = torch.full((A.MLP_PARAMS,), float("nan"), device=dev)
        A.mlp_backward(Wd, cache, dY, dW)
        out.append(dW.cpu().numpy())
    assert np.array_equal(out[0], out[1])
    assert np.max(np.abs(out[0] - go)) <= 1e-4 * np.max(np.abs(go))

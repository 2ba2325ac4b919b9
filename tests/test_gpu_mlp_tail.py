"""The rows that fill up the last tile of the network's backward add nothing, whatever the last row holds."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 32, 33, 250, 300])
@pytest.mark.parametrize("layer", [0, 1])
def test_infinite_activation_in_the_last_row(gpu, n, layer):
    import torch
    from paper_1212_3333_amd import learned
    amr = gpu
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((n, 12), device="cuda", generator=g)
    T = torch.rand(n, device="cuda", generator=g)
    W = learned.init_weights(1, "cuda")
    Y, H = amr.mlp_forward(X, W)
    H[n - 1, 64 * layer:64 * layer + 64] = 1.0
    H[n - 1, 64 * (1 - layer) + 7] = 1.0
    ref, _ = amr.mlp_backward(X, W, H, Y, T)
    H[n - 1, 64 * layer + 9] = float("inf")
    dW, _ = amr.mlp_backward(X, W, H, Y, T)
    hit = torch.zeros_like(dW, dtype=torch.bool)
    if layer:
        hit[4992 + 2 * 9:4992 + 2 * 9 + 2] = True             # dW3 of the unit
    else:
        hit[832 + 64 * 9:832 + 64 * 10] = True                # dW2 of the unit
    # dW2 of a unit that layer 2 cuts off in that row is inf x 0 by the definition
    assert torch.isinf(dW[hit]).any() and (layer == 0 or torch.isinf(dW[hit]).all())
    if layer == 0:
        cut = H[n - 1, 64:] <= 0
        assert torch.isnan(dW[hit][cut]).all() and torch.isinf(dW[hit][~cut]).all()
    assert torch.isfinite(dW[~hit]).all() and float((dW[~hit] - ref[~hit]).abs().max()) <= 1e-6 * float(ref.abs().max())

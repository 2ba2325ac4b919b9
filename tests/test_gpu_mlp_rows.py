"""The network's kernels at row counts around a tile of 32 rows, a block's eight tiles and the backward's
grid, and with arrays aligned to 4 bytes only.  A row's outputs depend on no other row: bit for bit.
The gradient is the mean over rows: that of n rows equals the weighted mean of two parts' gradients,
each of whose terms the kernels round to fp16 in at most three places (2^-11 each: 1.5e-3 together,
2e-3 allowed, in norm); the loss is summed in fp32."""
import pytest

from paper_1212_3333_amd import _stream, _vp
from paper_1212_3333_amd._lib import check, load

pytestmark = pytest.mark.gpu


def _inputs(n, seed):
    import torch
    from paper_1212_3333_amd import learned
    g = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randn((n, 12), device="cuda", generator=g)
    T = torch.rand(n, device="cuda", generator=g)
    return X, T, learned.init_weights(seed, "cuda")


def _off(t):
    """The same values at an address that is a multiple of 4 bytes only."""
    import torch
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)[1:]
    return buf.view(t.shape).copy_(t)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 255, 256, 257, 4097])
def test_rows(gpu, n):
    import torch
    amr = gpu
    X, T, W = _inputs(n, n)
    Y, H = amr.mlp_forward(X, W)
    a = max(n // 3, 1)
    for lo, hi in ((0, a), (a, n)):
        if hi > lo:
            y, h = amr.mlp_forward(X[lo:hi].contiguous(), W)
            assert torch.equal(y, Y[lo:hi]) and torch.equal(h, H[lo:hi])
    y0, _ = amr.mlp_forward(X, W, keep_hidden=False)
    assert torch.equal(y0, Y)
    dW, loss = amr.mlp_backward(X, W, H, Y, T)
    assert torch.isfinite(dW).all()
    if n > 1:
        parts = [amr.mlp_backward(X[s].contiguous(), W, H[s].contiguous(), Y[s].contiguous(), T[s].contiguous())
                 for s in (slice(0, a), slice(a, n))]
        w = (a / n, (n - a) / n)
        ref = sum(k * p[0].double() for k, p in zip(w, parts))
        assert float((dW.double() - ref).norm() / ref.norm()) <= 2e-3
        assert abs(float(loss) - sum(k * float(p[1]) for k, p in zip(w, parts))) <= 1e-5 * float(loss)


@pytest.mark.parametrize("n", [33, 300])
def test_four_byte_alignment(gpu, n):
    import torch
    amr = gpu
    X, T, W = _inputs(n, 7)
    Y, H = amr.mlp_forward(X, W)
    dW, loss = amr.mlp_backward(X, W, H, Y, T)
    x, t, w = _off(X), _off(T), _off(W)
    y, h, dw, ls = _off(torch.zeros_like(Y)), _off(torch.zeros_like(H)), _off(torch.zeros_like(W)), _off(torch.zeros(1, device="cuda"))
    assert h.data_ptr() % 16 == 4
    lib, st = load(), _stream(X.device)
    check(lib.amr_mlp_forward(_vp(x), _vp(w), _vp(y), _vp(h), n, st), "amr_mlp_forward")
    check(lib.amr_mlp_backward(_vp(x), _vp(w), _vp(h), _vp(y), _vp(t), n, 0.01, 0.99, _vp(dw), _vp(ls), st), "amr_mlp_backward")
    torch.cuda.synchronize()
    assert torch.equal(y, Y) and torch.equal(h, H)
    assert float((dw - dW).norm() / dW.norm()) <= 1e-5 and abs(float(ls) - float(loss)) <= 1e-5 * float(loss)

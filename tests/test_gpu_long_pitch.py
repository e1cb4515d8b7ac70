"""GPU parity, exact, of the register-staged kernel, which takes operands with a row pitch of 16 MB and more: the three operand layouts,
both operand types, and its epilogues.  Small integers: sums stay below 2^24, so the FP32 product of torch is exact too."""
import pytest
import torch

import paper_2303_11257_amd as us
from gpu_util import DEV, ptr, stream

pytestmark = pytest.mark.gpu
LONG = {False: 1 << 23, True: 1 << 24}          # elements of FP16 / FP8 in 16 MB


def _ints(shape, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randint(-2, 3, shape, generator=g, device=DEV, dtype=torch.int8).to(torch.float16)


def _operand(x, fp8, fmt):
    if not fp8:
        return x
    y = torch.empty(x.shape, dtype=torch.uint8, device=DEV)
    us.cast_fp8(ptr(x), us.F16, ptr(y), fmt, x.numel(), 1.0, None, stream())
    return y


def _layer(b, m, n, fp8, which):
    fmt = dict(X=us.E4M3, W=us.E4M3, G=us.E5M2)
    ints = {k: _ints(s, i) for i, (k, s) in enumerate(dict(X=(b, m), W=(m, n), G=(b, n)).items()) if k in which}
    dt = tuple(fmt.values()) if fp8 else (us.F16,) * 3
    return [ints[k] for k in which], [_operand(ints[k], fp8, fmt[k]) for k in which], dt


def _half(x, s):
    return (x * s).to(torch.float16)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("long_dim", ["m", "n"])
def test_forward_with_activation(long_dim, fp8):
    b, m, n = (48, LONG[fp8], 16) if long_dim == "m" else (48, 16, LONG[fp8])
    (X, W), (Xo, Wo), dt = _layer(b, m, n, fp8, "XW")
    Y, H = (torch.empty((b, n), dtype=torch.float16, device=DEV) for _ in range(2))
    s = 2.0 ** -12 if long_dim == "m" else 2.0 ** -3
    us.linear_fwd(ptr(Xo), ptr(Wo), ptr(Y), b, m, n, dt[0], dt[1], us.F16, s, us.EPI_GELU | us.EPI_ACT_RELU, 1.0, ptr(H), None, None, 0, stream())
    assert "staged" in us.last_launch()
    want = _half(X.float() @ W.float(), s)
    assert torch.equal(Y, want) and torch.equal(H, want.clamp_min(0))


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("epi", ["plain", "relu", "residual"])
def test_grad_x(epi, fp8):
    b, m, n = 16, 48, LONG[fp8]
    (W, G), (Wo, Go), dt = _layer(b, m, n, fp8, "WG")
    dX, z = torch.empty((b, m), dtype=torch.float16, device=DEV), torch.randn((b, m), device=DEV).to(torch.float16)
    code, scale = {"plain": (us.EPI_NONE, 0.0), "relu": (us.EPI_GELU_GRAD | us.EPI_ACT_RELU, 1.0), "residual": (us.EPI_RESIDUAL, 0.6)}[epi]
    us.linear_bwd(None, ptr(Wo), ptr(Go), ptr(dX), None, b, m, n, *dt, us.F16, 2.0 ** -12, 0.0, code, scale, ptr(z) if epi != "plain" else None,
                  None, None, 0, stream())
    assert "staged" in us.last_launch()
    d = _half(G.float() @ W.float().t().contiguous(), 2.0 ** -12)
    if epi == "residual":              # one rounding to FP16 of a sum of two products
        want = 0.8 * z.float() + 0.6 * d.float()
        assert bool(((dX.float() - want).abs() <= 2.0 ** -10 * want.abs() + 2.0 ** -20).all())
    else:
        assert torch.equal(dX, d if epi == "plain" else torch.where(z > 0, d, torch.zeros_like(d)))


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("long_dim", ["m", "n"])
def test_grad_w(long_dim, fp8):
    b, m, n = (48, LONG[fp8], 16) if long_dim == "m" else (48, 16, LONG[fp8])
    (X, G), (Xo, Go), dt = _layer(b, m, n, fp8, "XG")
    dW = torch.empty((m, n), dtype=torch.float16, device=DEV)
    wsb = us.workspace_bytes(b, m, n)
    assert wsb == us.TABLE_AREA_BYTES                  # no K slices
    us.linear_bwd(ptr(Xo), None, ptr(Go), None, ptr(dW), b, m, n, *dt, us.F16, 0.0, 2.0 ** -3, us.EPI_NONE, 0.0, None, None, None, 0, stream())
    assert "staged" in us.last_launch()
    assert torch.equal(dW, _half(X.float().t().contiguous() @ G.float(), 2.0 ** -3))

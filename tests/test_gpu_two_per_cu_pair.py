"""GPU parity, exact, of a layer's two backward products on four-wave 128 x 128 tiles, two workgroups per CU, in one launch: the edges of
its window (two tiles on every CU, few tiles, short and ragged reductions), every epilogue of grad_X and both operand types, and the
layers just beside the window.  Small integers: sums stay below 2^24, so the FP32 product of torch is exact too."""
import pytest
import torch

import paper_2303_11257_amd as us
from gpu_util import DEV, ptr, stream

pytestmark = pytest.mark.gpu
PAIR = "pair:128x128:wk1:st2:{p}:NT:{e}:s1 + pair:128x128:wk1:st2:{p}:TN:store:s1"


def _operands(b, m, n, fp8):
    out, dt = [], []
    for i, (shape, fmt) in enumerate((((b, m), us.E4M3), ((m, n), us.E4M3), ((b, n), us.E5M2))):
        x = torch.randint(-2, 3, shape, generator=torch.Generator(device=DEV).manual_seed(b + i), device=DEV, dtype=torch.int8).to(torch.float16)
        y = x
        if fp8:
            y = torch.empty(shape, dtype=torch.uint8, device=DEV)
            us.cast_fp8(ptr(x), us.F16, ptr(y), fmt, x.numel(), 1.0, None, stream())
        out.append((x, y))
        dt.append(fmt if fp8 else us.F16)
    return out, dt


def _bwd(b, m, n, fp8, epi):
    ((X, Xo), (W, Wo), (G, Go)), dt = _operands(b, m, n, fp8)
    z = torch.randn((b, m), device=DEV).to(torch.float16)
    dX, dW, dX8 = torch.full_like(z, 7.0), torch.full_like(W, 7.0), torch.empty((b, m), dtype=torch.uint8, device=DEV)
    ws = torch.full((us.workspace_bytes(b, m, n),), 0x5A, dtype=torch.uint8, device=DEV)
    code, scale = {"plain": (us.EPI_NONE, 0.0), "relu": (us.EPI_GELU_GRAD | us.EPI_ACT_RELU, 1.0), "residual": (us.EPI_RESIDUAL, 0.6)}[epi]
    sx, sw = 2.0 ** -6, 2.0 ** -6
    us.linear_bwd(ptr(Xo), ptr(Wo), ptr(Go), ptr(dX), ptr(dW), b, m, n, *dt, us.F16, sx, sw, code, scale, ptr(z) if epi != "plain" else None,
                  ptr(dX8) if epi == "relu" else None, ptr(ws), ws.numel(), stream())
    rec = us.last_launch()
    assert torch.equal(dW, (X.float().t().contiguous() @ G.float() * sw).to(torch.float16)), rec
    d = (G.float() @ W.float().t().contiguous() * sx).to(torch.float16)
    if epi == "residual":              # one rounding to FP16 of a sum of two products
        want = 0.8 * z.float() + 0.6 * d.float()
        assert bool(((dX.float() - want).abs() <= 2.0 ** -10 * want.abs() + 2.0 ** -20).all()), rec
    else:
        assert torch.equal(dX, d if epi == "plain" else torch.where(z > 0, d, torch.zeros_like(d))), rec
    if epi == "relu":
        want8 = torch.empty_like(dX8)
        us.cast_fp8(ptr(dX), us.F16, ptr(want8), us.E5M2, dX.numel(), 1.0, None, stream())
        assert torch.equal(dX8, want8), rec
    return rec


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("epi", ["plain", "relu", "residual"])
@pytest.mark.parametrize("b,m,n", [(2048, 2048, 2032), (640, 3328, 512), (656, 3344, 528), (2688, 768, 2304), (5504, 864, 2704), (896, 4528, 752)])
def test_pair_is_exact(b, m, n, epi, fp8):
    p, e = "fp8" if fp8 else "f16", {"plain": "store", "relu": "act_grad", "residual": "residual"}[epi]
    assert _bwd(b, m, n, fp8, epi) == PAIR.format(p=p, e=e)


@pytest.mark.parametrize("fp8", [False, True])
def test_ragged_pair_with_activation(fp8):
    assert _bwd(2000, 1552, 2064, fp8, "relu").startswith("pair:128x128:wk1:st2")


W128 = "pair:128x128:wk2:st4:"
# layer -> the grad_X kernel that it takes instead
# (None: the pair of this file)
@pytest.mark.parametrize("b,m,n,epi,fp8,grad_x", [(2000, 1552, 2064, "plain", False, W128),     # plain, fewer than seven tiles per four CUs
                                                  (2000, 1552, 2064, "plain", True, W128),
                                                  (2048, 1536, 2048, "residual", True, None),   # ... which holds without an epilogue only
                                                  (1232, 1392, 1632, "relu", False, W128),      # eight-wave tiles fit one round
                                                  (1232, 1392, 1632, "relu", True, W128),
                                                  (2320, 816, 3536, "relu", False, W128),       # ... with long grad_W tiles
                                                  (3536, 1056, 976, "relu", False, "direct:"),  # few grad_W tiles with a long reduction
                                                  (1664, 2304, 2048, "relu", False, "direct:")])  # more tiles than resident at once
def test_beside_the_window(b, m, n, epi, fp8, grad_x):
    rec = _bwd(b, m, n, fp8, epi)
    pair = PAIR.format(p="fp8" if fp8 else "f16", e={"plain": "store", "relu": "act_grad", "residual": "residual"}[epi])
    assert rec == pair if grad_x is None else rec != pair and rec.startswith(grad_x), rec


@pytest.mark.parametrize("fp8", [False, True])
def test_column_sums(fp8):
    """The bias gradient of an FFN whose second layer's backward pass takes this pair: the sums of the stored FP16 dZ."""
    T, d, f = 656, 528, 3344
    dt = torch.float16
    X, W1, W2, G, Z = (torch.randn(s, device=DEV).to(dt) for s in ((T, d), (d, f), (f, d), (T, d), (T, f)))
    ops = []
    for x, fmt in ((X, us.E4M3), (W1, us.E4M3), (W2, us.E4M3), (Z, us.E4M3), (G, us.E5M2)):
        y = x
        if fp8:
            y = torch.empty(x.shape, dtype=torch.uint8, device=DEV)
            us.cast_fp8(ptr(x), us.F16, ptr(y), fmt, x.numel(), 1.0, None, stream())
        ops.append(y)
    Xo, W1o, W2o, H, Go = ops
    dZ, dX, dW1, dW2 = torch.empty_like(Z), torch.empty_like(X), torch.empty_like(W1), torch.empty_like(W2)
    dZ8, db1, db2 = torch.empty((T, f), dtype=torch.uint8, device=DEV), torch.empty(f, dtype=dt, device=DEV), torch.empty(d, dtype=dt, device=DEV)
    ws = torch.empty(us.ffn_bias_workspace_bytes(T, d, f), dtype=torch.uint8, device=DEV)
    us.ffn_bias_bwd(ptr(Xo), ptr(W1o), ptr(W2o), ptr(Z), ptr(H), ptr(Go), ptr(G), ptr(dZ), ptr(dZ8) if fp8 else None, ptr(dX), ptr(dW1), ptr(dW2),
                    ptr(db1), ptr(db2), T, d, f, us.FFN_FP8 if fp8 else 0, ptr(ws), ws.numel(), stream())
    assert us.last_launch().startswith("pair:128x128:wk1:st2"), us.last_launch()
    want = dZ.double().sum(0) * T ** -0.5
    # FP32 sums of 656 values of about one, then one rounding to FP16
    assert bool(((db1.double() - want).abs() <= 2.0 ** -10 * want.abs() + 1e-5 * T ** 0.5).all())

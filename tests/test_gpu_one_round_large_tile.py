"""GPU parity, exact, of forward and grad_X products whose small tiles would need a second round on the CUs and whose large tiles fit one:
ragged in every dimension, both operand types, every kind of epilogue, and the products just beside the window.  Small integers: sums
stay below 2^24, so the FP32 product of torch is exact too."""
import pytest
import torch

import paper_2303_11257_amd as us
from gpu_util import DEV, ptr, stream

pytestmark = pytest.mark.gpu


def _operand(shape, fp8, fmt, seed):
    x = torch.randint(-2, 3, shape, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV, dtype=torch.int8).to(torch.float16)
    if not fp8:
        return x, x, us.F16
    y = torch.empty(shape, dtype=torch.uint8, device=DEV)
    us.cast_fp8(ptr(x), us.F16, ptr(y), fmt, x.numel(), 1.0, None, stream())
    return x, y, fmt


def _fwd(M, N, K, fp8, epi):
    (X, Xo, xd), (W, Wo, wd) = _operand((M, K), fp8, us.E4M3, 1), _operand((K, N), fp8, us.E4M3, 2)
    Y, H, skip = (torch.empty((M, N), dtype=torch.float16, device=DEV) for _ in range(3))
    ws = torch.empty(us.TABLE_AREA_BYTES, dtype=torch.uint8, device=DEV)
    us.gelu_tables(ptr(ws), ws.numel(), 0.0, 0.0, stream())
    bias = torch.randint(-2, 3, (N,), device=DEV).to(torch.float16) if epi == "bias" else None
    skip.normal_()
    code = {"plain": 0, "bias": 0, "relu": us.EPI_GELU | us.EPI_ACT_RELU, "gelu": us.EPI_GELU | us.EPI_TABLES_READY, "residual": us.EPI_RESIDUAL}[epi]
    us.linear_bias_fwd(ptr(Xo), ptr(Wo), ptr(bias), ptr(Y), M, K, N, xd, wd, us.F16, 2.0 ** -5, code, {"residual": 0.6, "relu": 1.0}.get(epi, 0.0),
                       ptr(skip) if epi == "residual" else ptr(H) if code else None, None, ptr(ws), ws.numel(), stream())
    rec, d = us.last_launch(), (X.float() @ W.float() * 2.0 ** -5)
    if epi == "residual":              # one rounding to FP16 of a sum of two products
        want = 0.8 * skip.float() + 0.6 * d.to(torch.float16).float()
        assert bool(((Y.float() - want).abs() <= 2.0 ** -10 * want.abs() + 2.0 ** -20).all()), rec
        return rec
    d = (d + bias.float() if epi == "bias" else d).to(torch.float16)
    assert torch.equal(Y, d), rec
    if epi == "relu":
        assert torch.equal(H, d.clamp_min(0)), rec
    if epi == "gelu":
        want = torch.empty_like(H)
        us.gelu_fwd(ptr(Y), ptr(want), Y.numel(), us.F16, 0.0, stream())
        assert torch.equal(H, want), rec
    return rec


def _dx(M, N, K, fp8, epi):
    (G, Go, gd), (W, Wo, wd) = _operand((M, K), fp8, us.E5M2, 3), _operand((N, K), fp8, us.E4M3, 4)
    dX, z = torch.empty((M, N), dtype=torch.float16, device=DEV), torch.randn((M, N), device=DEV).to(torch.float16)
    code = us.EPI_GELU_GRAD | us.EPI_ACT_RELU if epi == "relu" else 0
    us.linear_bwd(None, ptr(Wo), ptr(Go), ptr(dX), None, M, N, K, us.E4M3 if fp8 else us.F16, wd, gd, us.F16, 2.0 ** -5, 0.0, code, 1.0, ptr(z) if code else None,
                  None, None, 0, stream())
    rec, d = us.last_launch(), (G.float() @ W.float().t().contiguous() * 2.0 ** -5).to(torch.float16)
    assert torch.equal(dX, torch.where(z > 0, d, torch.zeros_like(d)) if code else d), rec
    return rec


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("epi", ["plain", "bias", "relu", "gelu", "residual"])
@pytest.mark.parametrize("M,N,K", [(3136, 2640, 784), (6000, 1552, 1504), (2048, 4224, 768), (17664, 496, 1040)])
def test_forward(M, N, K, epi, fp8):
    assert "direct:256x256:wk1" in _fwd(M, N, K, fp8, epi)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("epi", ["plain", "relu"])
@pytest.mark.parametrize("M,N,K", [(11936, 992, 784), (2080, 4272, 1232)])
def test_grad_x(M, N, K, epi, fp8):
    assert "direct:256x256:wk1" in _dx(M, N, K, fp8, epi)


@pytest.mark.parametrize("M,N,K", [(4096, 2048, 1024),         # as many small tiles as fit two per CU
                                   (3136, 2640, 368),          # a short reduction
                                   (4352, 4096, 1024)])        # more large tiles than CUs
def test_beside_the_window(M, N, K):
    assert "direct:128x128:wk1" in _fwd(M, N, K, False, "plain")


def _arithmetic_gelu(M, N, K, fp8, back, workspace):
    """The arithmetic GELU (both copies, which no table makes) or GELU' (no workspace to hold a table) of a call that says its tables are ready."""
    (A, Ao, ad), (B, Bo, bd) = _operand((M, K), fp8, us.E5M2 if back else us.E4M3, 5), _operand((N, K) if back else (K, N), fp8, us.E4M3, 6)
    Y, H, z = torch.empty((M, N), dtype=torch.float16, device=DEV), torch.empty((M, N), dtype=torch.float16, device=DEV), torch.randn((M, N), device=DEV).half()
    H8, want, want8 = torch.empty((M, N), dtype=torch.uint8, device=DEV), torch.empty_like(H), torch.empty((M, N), dtype=torch.uint8, device=DEV)
    ws = torch.empty(us.TABLE_AREA_BYTES if workspace else 0, dtype=torch.uint8, device=DEV)
    w = (ptr(ws) if workspace else None, ws.numel(), stream())
    if workspace:
        us.gelu_tables(ptr(ws), ws.numel(), 0.0, 0.0, stream())
    d = (A.float() @ (B.float().t().contiguous() if back else B.float()) * 2.0 ** -5).half()
    if back:
        us.linear_bwd(None, ptr(Bo), ptr(Ao), ptr(H), None, M, N, K, us.E4M3 if fp8 else us.F16, bd, ad, us.F16, 2.0 ** -5, 0.0,
                      us.EPI_GELU_GRAD | us.EPI_TABLES_READY, 0.0, ptr(z), ptr(H8), *w)
        rec = us.last_launch()
        us.gelu_bwd(ptr(z), ptr(d), ptr(want), d.numel(), us.F16, 0.0, stream())
    else:
        us.linear_fwd(ptr(Ao), ptr(Bo), ptr(Y), M, K, N, ad, bd, us.F16, 2.0 ** -5, us.EPI_GELU | us.EPI_TABLES_READY, 0.0, ptr(H), ptr(H8), *w)
        rec = us.last_launch()
        us.gelu_fwd(ptr(d), ptr(want), d.numel(), us.F16, 0.0, stream())
        assert torch.equal(Y, d)
    us.cast_fp8(ptr(H), us.F16, ptr(want8), us.E5M2 if back else us.E4M3, H.numel(), 1.0, None, stream())
    assert torch.equal(H, want) and torch.equal(H8, want8)
    return rec


@pytest.mark.parametrize("M,N,back,workspace,fp8", [(3136, 2640, False, True, False), (8672, 1008, False, False, False), (5296, 1952, True, False, False),
                                                    (5296, 1952, True, False, True)])
def test_arithmetic_gelu_needs_twice_the_reduction(M, N, back, workspace, fp8):
    """Whether or not the tables are said to be ready: 1536 bytes of reduction for the large tile, 16 values less for the small one."""
    K = 1536 if fp8 else 768
    for k, tile in ((K, "256x256"), (K - 16, "128x128"), (K // 2, "128x128")):
        rec = _arithmetic_gelu(M, N, k, fp8, back, workspace)
        assert f"direct:{tile}:wk1" in rec and ("act_grad" if back else ":act:") in rec

"""GPU parity of the few-tiles kernel (us_gemm_small.h) at the edges of its tiles and of its reduction split: outputs of one
ragged tile and of just as many tiles as CUs for each tile size, reductions with fewer stages than waves (64 bytes of K each),
one stage more than that, a cut last stage, and many stages per wave.  Operands are small integers and scales powers of two,
so the sum of the eight partial tiles is exact and must equal the oracle; the epilogues are compared with the same call's
plain result.  Tiles: 32 x 32, 32 x 64, 64 x 64 by the number of tiles, per us_gemm_dispatch.h."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2303_11257_amd as us
import synth
from gpu_util import DEV, assert_close, cast_fp8, empty, ptr, stream, to_dev

pytestmark = pytest.mark.gpu

# M, N, K of the product and its tile; every size is used in the three operand layouts
CASES = [
    (16, 16, 16, "32x32"), (16, 48, 32, "32x32"), (48, 80, 48, "32x32"), (64, 1024, 512, "32x32"), (496, 512, 528, "32x32"),
    (512, 512, 1040, "32x32"), (16, 4096, 2064, "32x32"), (528, 512, 240, "32x64"), (64, 4112, 112, "32x64"), (512, 1024, 3088, "32x64"),
    (528, 1008, 2064, "64x64"), (1024, 1024, 16, "64x64"), (1008, 1024, 1552, "64x64"), (80, 8192, 272, "64x64"),
]


def _problem(layout, M, N, K):
    """(b, m, n) of the layer whose product in this layout is M x N over K."""
    return {"fwd": (M, K, N), "dx": (M, N, K), "dw": (K, M, N)}[layout]


def _operands(b, m, n, fp8, seed):
    fmts = (us.E4M3, us.E4M3, us.E5M2) if fp8 else (us.F16,) * 3
    ints = [synth.small_ints(seed, t, s) for t, s in ((1, (b, m)), (2, (m, n)), (4, (b, n)))]
    return [cast_fp8(a, f) if fp8 else a for a, f in zip(ints, fmts)], fmts


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("layout", ["fwd", "dx", "dw"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:3])))
def test_exact(case, layout, fp8):
    M, N, K, tile = case
    b, m, n = _problem(layout, M, N, K)
    (X, W, G), dt = _operands(b, m, n, fp8, 900 + M + N + K)
    odt = (O.E4M3, O.E4M3, O.E5M2) if fp8 else (O.F16,) * 3
    tX, tW, tG = to_dev(X), to_dev(W), to_dev(G)
    wsb = us.workspace_bytes(b, m, n)
    ws = torch.full((wsb,), 0x5A, dtype=torch.uint8, device=DEV)
    s = 2.0 ** -4
    for out_dt, odt_out, np_dt in ((us.F16, O.F16, np.float16), (us.F32, O.F32, np.float32)):
        C = torch.full((M * N + 64,), 7.0, dtype=torch.float16 if np_dt == np.float16 else torch.float32, device=DEV)
        if layout == "fwd":
            us.linear_fwd(ptr(tX), ptr(tW), ptr(C), b, m, n, dt[0], dt[1], out_dt, s, us.EPI_NONE, 0.0, None, None, None, 0, stream())
            ref = O.linear_fwd(X, W, s, odt[0], odt[1], odt_out)
        else:
            dX, dW = (C, None) if layout == "dx" else (None, C)
            us.linear_bwd(ptr(tX), ptr(tW), ptr(tG), ptr(dX), ptr(dW), b, m, n, *dt, out_dt, s, s, us.EPI_NONE, 0.0, None, None, ptr(ws), wsb,
                          stream())
            ref = O.linear_bwd_dx(G, W, s, odt[2], odt[1], odt_out) if layout == "dx" else O.linear_bwd_dw(X, G, s, odt[0], odt[2], odt_out)
        assert f"direct:{tile}:wk8" in us.last_launch(), us.last_launch()
        got = C.cpu().numpy()
        assert np.all(got[M * N:] == 7.0)
        assert np.array_equal(got[:M * N].reshape(M, N), ref)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("shape", [(16, 48, 80), (496, 528, 512), (528, 1008, 272), (1008, 272, 1024)], ids=lambda s: "x".join(map(str, s)))
def test_epilogues(shape, fp8):
    """Bias, every activation with its copies, the residual interpolation, every activation derivative, from the plain result."""
    b, m, n = shape
    (X, W, G), dt = _operands(b, m, n, fp8, 950 + b)
    tX, tW, tG = to_dev(X), to_dev(W), to_dev(G)
    bias, skip, zpre = synth.normal(951, 9, (n,)), synth.normal(952, 10, (b, n)), synth.normal(953, 11, (b, m))
    tb, ts, tz = to_dev(bias), to_dev(skip), to_dev(zpre)
    st = stream()
    Y, Yb, Out, Z, H, dX, dZ = (empty(s, np.float16) for s in ((b, n),) * 5 + ((b, m),) * 2)
    H8, dZ8 = empty((b, n), np.uint8), empty((b, m), np.uint8)
    fwd = lambda f, *a: f(ptr(tX), ptr(tW), *a)
    us.linear_fwd(ptr(tX), ptr(tW), ptr(Y), b, m, n, dt[0], dt[1], us.F16, 0.0, us.EPI_NONE, 0.0, None, None, None, 0, st)
    us.linear_bias_fwd(ptr(tX), ptr(tW), ptr(tb), ptr(Yb), b, m, n, dt[0], dt[1], us.F16, 0.0, us.EPI_NONE, 0.0, None, None, None, 0, st)
    us.linear_fwd(ptr(tX), ptr(tW), ptr(Out), b, m, n, dt[0], dt[1], us.F16, 0.0, us.EPI_RESIDUAL, 0.6, ptr(ts), None, None, 0, st)
    us.linear_bwd(None, ptr(tW), ptr(tG), ptr(dX), None, b, m, n, *dt, us.F16, 0.0, 0.0, us.EPI_NONE, 0.0, None, None, None, 0, st)
    assert ":wk8:" in us.last_launch()
    y, odt = Y.cpu().numpy(), (O.E4M3, O.E4M3) if fp8 else (O.F16, O.F16)
    assert_close(Yb.cpu().numpy(), O.linear_fwd(X, W, O.linear_scales(b, m, n)[0], *odt, bias=bias), "Y + bias", fp8=fp8)
    sw = np.float32(np.sqrt(1 - np.float32(0.6) ** 2))
    assert_close(Out.cpu().numpy(), O.weighted_add2(skip, y, sw, np.float32(0.6)), "residual")
    for act in (0, us.EPI_ACT_RELU, us.EPI_ACT_TANH, us.EPI_ACT_SIGMOID):
        us.linear_fwd(ptr(tX), ptr(tW), ptr(Z), b, m, n, dt[0], dt[1], us.F16, 0.0, us.EPI_GELU | act, 0.0, ptr(H), ptr(H8), None, 0, st)
        us.linear_bwd(None, ptr(tW), ptr(tG), ptr(dZ), None, b, m, n, *dt, us.F16, 0.0, 0.0, us.EPI_GELU_GRAD | act, 0.0, ptr(tz), ptr(dZ8),
                      None, 0, st)
        assert ":wk8:" in us.last_launch()
        assert np.array_equal(Z.cpu().numpy(), y)
        want = empty((b, n), np.float16), empty((b, m), np.float16)
        us.act_fwd(ptr(Y), ptr(want[0]), b * n, us.F16, act >> 4, 0.0, 0.0, st)
        us.act_bwd(ptr(tz), ptr(dX), ptr(want[1]), b * m, us.F16, act >> 4, 0.0, 0.0, st)
        assert torch.equal(H, want[0]) and torch.equal(dZ, want[1])
        assert np.array_equal(H8.cpu().numpy(), O.cast_fp8(H.cpu().numpy(), O.E4M3)[0])
        assert np.array_equal(dZ8.cpu().numpy(), O.cast_fp8(dZ.cpu().numpy(), O.E5M2)[0])


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("shape,tile", [((16, 16, 48), "32x32"), ((272, 256, 1024), "32x32"), ((1040, 272, 1024), "32x64"),
                                        ((528, 1008, 1024), "64x64"), ((2000, 80, 16), "32x32")], ids=str)
def test_backward_in_one_launch(shape, tile, fp8):
    """grad_X and grad_W together equal the two products alone, plain (integers: bit for bit) and with the activation derivative;
    a grad_W that overwrites the weights comes after grad_X has read them."""
    b, m, n = shape
    (X, W, G), dt = _operands(b, m, n, fp8, 970 + b)
    tX, tW, tG, tz = to_dev(X), to_dev(W), to_dev(G), to_dev(synth.normal(971, 11, (b, m)))
    wsb = us.workspace_bytes(b, m, n)
    ws = torch.full((wsb,), 0x5A, dtype=torch.uint8, device=DEV)
    s = 2.0 ** -4

    def bwd(dX, dW, epi=us.EPI_NONE, z=None, W_=tW):
        us.linear_bwd(ptr(tX), ptr(W_), ptr(tG), ptr(dX), ptr(dW), b, m, n, *dt, us.F16, s, s, epi, 0.5 if epi == us.EPI_RESIDUAL else 0.0,
                      ptr(z), None, ptr(ws), wsb, stream())
        return us.last_launch()
    e = lambda: (empty((b, m), np.float16), empty((m, n), np.float16))
    for epi in (us.EPI_NONE, us.EPI_GELU_GRAD, us.EPI_GELU_GRAD | us.EPI_ACT_TANH, us.EPI_RESIDUAL):
        z = tz if epi != us.EPI_NONE else None
        (dX, dW), (dX1, dW1) = e(), e()
        rec = bwd(dX, dW, epi, z)
        assert rec.count(f"pair:{tile}:wk8") == 2, rec
        bwd(dX1, None, epi, z), bwd(None, dW1, epi, z)
        assert torch.equal(dX, dX1) and torch.equal(dW, dW1)
    (dX1, dW1), Wcopy = e(), torch.zeros((2 * m * n,), dtype=torch.uint8, device=DEV)
    Wcopy[:tW.numel() * tW.element_size()] = tW.view(torch.uint8).flatten()
    assert "pair" not in bwd(dX1, Wcopy, W_=Wcopy)
    bwd(dX, dW)
    assert torch.equal(dX, dX1) and torch.equal(dW.view(torch.uint8).flatten(), Wcopy)

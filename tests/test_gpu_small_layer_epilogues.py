"""GPU parity of the epilogues on the 128 x 128 tile of eight waves and on the 128 x 256 tile of FP8 forward products, with ragged rows,
columns and reduction: bias, every activation with its copies, the residual interpolation and every activation derivative.
Small integers: the plain result is exact, and each epilogue must agree with the stand-alone operation on it.  And the lines
between which a product takes the 128 x 256 tile."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2303_11257_amd as us
import synth
from gpu_util import DEV, assert_close, cast_fp8, empty, ptr, stream, to_dev

pytestmark = pytest.mark.gpu
ACTS = (0, us.EPI_ACT_RELU, us.EPI_ACT_TANH, us.EPI_ACT_SIGMOID)


class _Layer:
    def __init__(self, b, m, n, fp8):
        ops = [synth.small_ints(960 + b, t, s) for t, s in ((1, (b, m)), (2, (m, n)), (4, (b, n)))]
        self.dt = (us.E4M3, us.E4M3, us.E5M2) if fp8 else (us.F16,) * 3
        self.shape, (self.X, self.W, self.G) = (b, m, n), (to_dev(cast_fp8(a, f) if fp8 else a) for a, f in zip(ops, self.dt))

    def fwd(self, Y, epi=us.EPI_NONE, scale=0.0, a16=None, a8=None, bias=None):
        us.linear_bias_fwd(ptr(self.X), ptr(self.W), ptr(bias), ptr(Y), *self.shape, self.dt[0], self.dt[1], us.F16, 2.0 ** -6, epi, scale,
                           ptr(a16), ptr(a8), None, 0, stream())
        return us.last_launch()

    def dx(self, dX, epi=us.EPI_NONE, scale=0.0, z=None, a8=None):
        us.linear_bwd(None, ptr(self.W), ptr(self.G), ptr(dX), None, *self.shape, *self.dt, us.F16, 2.0 ** -6, 0.0, epi, scale, ptr(z), ptr(a8),
                      None, 0, stream())
        return us.last_launch()


@pytest.mark.parametrize("shape,fp8,fwd,dx", [((1040, 1936, 1552), False, "128x128:wk2:st4", "128x128:wk2:st4"),
                                              ((1040, 1936, 1552), True, "128x128:wk2:st4", "128x128:wk2:st4"),
                                              ((2000, 1552, 2064), True, "128x256:wk1", None)], ids=str)
def test_epilogues(shape, fp8, fwd, dx):
    b, m, n = shape
    L = _Layer(b, m, n, fp8)
    st, h = stream(), np.float16
    Y, Yb, R, Z, H, want, H8 = *(empty((b, n), h) for _ in range(6)), empty((b, n), np.uint8)
    bias, skip, zpre = to_dev(synth.normal(961, 9, (n,))), to_dev(synth.normal(962, 10, (b, n))), to_dev(synth.normal(963, 11, (b, m)))
    runs = [L.fwd(Y), L.fwd(Yb, bias=bias), L.fwd(R, us.EPI_RESIDUAL, 0.6, skip)]
    # (integers times 2^-6 below 2^5 are exact in FP16)
    assert float(Y.float().abs().max()) < 32.0 and torch.equal(Yb, (Y.float() + bias.float()).to(torch.float16))
    assert_close(R.cpu().numpy(), O.weighted_add2(skip.cpu().numpy(), Y.cpu().numpy(), np.float32(np.sqrt(1 - np.float32(0.6) ** 2)),
                                                  np.float32(0.6)), "residual")
    for act in ACTS:
        runs.append(L.fwd(Z, us.EPI_GELU | act, 0.0, H, H8))
        us.act_fwd(ptr(Y), ptr(want), b * n, us.F16, act >> 4, 0.0, 0.0, st)
        assert torch.equal(Z, Y) and torch.equal(H, want)
        assert np.array_equal(H8.cpu().numpy(), O.cast_fp8(H.cpu().numpy(), O.E4M3)[0])
    assert all(fwd in r for r in runs), runs
    if dx is None:
        return
    dX, dZ, want, dZ8 = *(empty((b, m), h) for _ in range(3)), empty((b, m), np.uint8)
    runs = [L.dx(dX)]
    for act in ACTS:
        runs.append(L.dx(dZ, us.EPI_GELU_GRAD | act, 0.0, zpre, dZ8))
        us.act_bwd(ptr(zpre), ptr(dX), ptr(want), b * m, us.F16, act >> 4, 0.0, 0.0, st)
        assert torch.equal(dZ, want)
        assert np.array_equal(dZ8.cpu().numpy(), O.cast_fp8(dZ.cpu().numpy(), O.E5M2)[0])
    assert all(dx in r for r in runs), runs


@pytest.mark.parametrize("shape,wide", [((2112, 1552, 2048), True), ((2080, 1552, 2048), False), ((2112, 1664, 2048), False), ((2112, 1008, 2048), False),
                                        ((4160, 3072, 1024), True), ((4112, 3072, 1024), False), ((5632, 3072, 768), False)], ids=str)
def test_where_the_wide_tile_pays(shape, wide):
    """FP8 forward on both sides of each line, exact."""
    b, m, n = shape
    L = _Layer(b, m, n, True)
    Y = empty((b, n), np.float16)
    rec = L.fwd(Y)
    assert ("128x256" in rec) == wide, rec
    codes = lambda t, rows: t[rows].cpu().numpy()
    rows = torch.cat([torch.arange(0, b, 61, device=DEV), torch.tensor([b - 1], device=DEV)])
    assert np.array_equal(codes(Y, rows), O.linear_fwd(codes(L.X, rows), L.W.cpu().numpy(), 2.0 ** -6, O.E4M3, O.E4M3, O.F16))

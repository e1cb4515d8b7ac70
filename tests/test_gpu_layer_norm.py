"""GPU parity: scaled layer norm forward / backward against the oracle (Table A.2 "Other")."""
import numpy as np
import pytest
import torch

import oracle
import paper_2303_11257_amd as us
import synth
from gpu_util import DEV, assert_close, empty, ptr, stream, to_dev, to_np

pytestmark = pytest.mark.gpu
O = oracle


def _inputs(b, n, seed, sigma=1.0, shift=0.0):
    X = (synth.normal(seed, 1, (b, n), sigma=sigma).astype(np.float32) + shift).astype(np.float16)
    w = (1.0 + 0.25 * synth.normal(seed, 2, (n,)).astype(np.float32)).astype(np.float16)
    c = (0.1 * synth.normal(seed, 3, (n,)).astype(np.float32)).astype(np.float16)
    G = synth.normal(seed, 4, (b, n))
    return X, w, c, G


def _run(X, w, c, G, eps, beta=0.0):
    b, n = X.shape
    tX, tw, tc, tG = to_dev(X), to_dev(w), to_dev(c), to_dev(G)
    Y, dX, dw, dc = empty((b, n), np.float16), empty((b, n), np.float16), empty((n,), np.float16), empty((n,), np.float16)
    us.layer_norm_fwd(ptr(tX), ptr(tw), ptr(tc), ptr(Y), b, n, eps, stream())
    wsb = us.layer_norm_workspace_bytes(b, n)
    ws = torch.full((wsb,), 0x5A, dtype=torch.uint8, device=DEV)
    us.layer_norm_bwd(ptr(tX), ptr(tw), ptr(tG), ptr(dX), ptr(dw), ptr(dc), b, n, eps, beta, ptr(ws), wsb, stream())
    return to_np(Y), to_np(dX), to_np(dw), to_np(dc)


def _key(x):
    u = x.view(np.uint16).astype(np.int32)
    return np.where(u & 0x8000, -(u & 0x7fff), u)


@pytest.mark.parametrize("shape", [(1, 16), (50, 48), (272, 400), (1000, 768), (512, 1024), (131, 2064), (64, 4096), (140001, 16), (16432, 528)])
@pytest.mark.parametrize("eps", [0.0, 1e-5])
def test_forward_and_backward_against_the_oracle(shape, eps):
    """Row lengths below, at and across the 512-element wave chunk; row counts that are not multiples of the
    32-row blocks of the backward pass.  FP32 statistics against double: at most one FP16 step, rarely."""
    b, n = shape
    X, w, c, G = _inputs(b, n, 181 + n, sigma=1.7, shift=0.4)
    if n == 16 and eps == 0.0:
        X[0, :] = np.arange(16, dtype=np.float16)             # a row that certainly has spread
    Y, dX, dw, dc = _run(X, w, c, G, eps)
    rY, _, _ = O.layer_norm_fwd(X, w, c, eps)
    rdX, rdw, rdc = O.layer_norm_bwd(X, w, G, eps)
    assert int(np.max(np.abs(_key(Y) - _key(rY)))) <= 1 and np.mean(Y != rY) < 5e-3
    assert_close(dX, rdX, "dX")
    assert np.mean(dX != rdX) < 0.02
    assert_close(dw, rdw, "dw")
    assert_close(dc, rdc, "dc")


def test_bert_large_shape_variances_and_determinism():
    """b = 8192 tokens, n = 1024: unit weights, N(0,1) input and gradient.  Var(Y) = 1, Var(dX) = 1 - 2/n,
    Var(dw) = Var(dc) = 1 with the default b^-1/2; two runs are bit-identical (ordered block sums)."""
    b, n = 8192, 1024
    X, _, _, G = _inputs(b, n, 191)
    one, zero = np.ones(n, np.float16), np.zeros(n, np.float16)
    Y, dX, dw, dc = _run(X, one, zero, G, 0.0)
    v = lambda a: float(np.var(a.astype(np.float64)))
    assert abs(v(Y) - 1.0) < 0.01 and abs(v(dX) - (1 - 2 / n)) < 0.01
    assert abs(v(dw) - 1.0) < 0.12 and abs(v(dc) - 1.0) < 0.12
    rows = [0, 31, 32, 4095, 8191]
    rY, _, _ = O.layer_norm_fwd(X[rows], one, zero)
    assert int(np.max(np.abs(_key(Y[rows]) - _key(rY)))) <= 1
    cols = slice(0, 64)
    _, rdw, rdc = O.layer_norm_bwd(np.ascontiguousarray(X), one, G)
    assert_close(dw, rdw, "dw") and assert_close(dc, rdc, "dc")
    Y2, dX2, dw2, dc2 = _run(X, one, zero, G, 0.0)
    assert np.array_equal(dw, dw2) and np.array_equal(dc, dc2) and np.array_equal(dX, dX2)
    # an explicit weight-gradient scale
    _, _, dw3, _ = _run(X, one, zero, G, 0.0, beta=0.5)
    assert_close(dw3, O.layer_norm_bwd(X, one, G, 0.0, 0.5)[1], "dw, beta given")


def test_zero_variance_row_and_empty_input():
    X = np.full((4, 32), 3.0, np.float16)
    X[1] = np.arange(32, dtype=np.float16)
    w, c, G = np.ones(32, np.float16), np.full(32, 0.5, np.float16), np.ones((4, 32), np.float16)
    Y, _, _, _ = _run(X, w, c, G, 0.0)
    assert np.isnan(Y[0].astype(np.float32)).all() and np.isfinite(Y[1].astype(np.float32)).all()     # 0 * inf, as the formula says
    Y, _, _, _ = _run(X, w, c, G, 1e-5)
    assert np.all(Y[0] == np.float16(0.5))
    us.layer_norm_fwd(None, None, None, None, 0, 32, 0.0, stream())


@pytest.mark.parametrize("shape", [(1, 1040), (9, 1552), (33, 2048), (8192, 1040), (8193, 1040)])
def test_rows_of_three_and_four_chunks(shape):
    """Rows of 1032 to 2048 values, with fewer rows than waves, one block of 32 rows per CU and one more (8192 and 8193 rows), a last block of
    one row and a last chunk that few lanes have.  Bounds as above."""
    b, n = shape
    X, w, c, G = _inputs(b, n, 211 + n, sigma=1.7, shift=0.4)
    Y, dX, dw, dc = _run(X, w, c, G, 1e-5)
    rY, _, _ = O.layer_norm_fwd(X, w, c, 1e-5)
    rdX, rdw, rdc = O.layer_norm_bwd(X, w, G, 1e-5)
    assert int(np.max(np.abs(_key(Y) - _key(rY)))) <= 1 and np.mean(Y != rY) < 5e-3
    assert_close(dX, rdX, "dX")
    assert np.mean(dX != rdX) < 0.02
    assert_close(dw, rdw, "dw")
    assert_close(dc, rdc, "dc")


def _wave_sum(v):
    """64 lanes in pairs, then pairs of pairs, ...: [..., 64] -> [...]."""
    while v.shape[-1] > 1:
        v = v[..., 0::2] + v[..., 1::2]
    return v[..., 0]


def _fp32_layer_norm(X, w, c, G, eps, waves):
    """Both passes as the kernels round them: FP32, every product and every sum of the statistics and of the gradients rounded by itself (only
    the forward result is one fused multiply-add), in the order of the elements of a lane, the lanes of a row, the rows of a wave, the
    waves of a 32-row block and the blocks of one of 16 segments."""
    f = np.float32
    b, n = X.shape
    nch = -(-n // 512)
    lanes = lambda a: np.pad(a.astype(f), ((0, 0), (0, nch * 512 - n))).reshape(a.shape[0], nch, 64, 8)
    valid = (np.arange(nch * 512) < n).reshape(1, nch, 64, 8)
    rows = lambda a: a.reshape(b, nch * 512)[:, :n]

    def row_sum(t):
        s = np.zeros((b, 64), f)
        for k in range(nch):
            for e in range(8):
                s = s + np.where(valid[:, k, :, e], t[:, k, :, e], f(0))
        return _wave_sum(s)[:, None, None, None]

    x, g, wr = lanes(X), lanes(G), lanes(w[None])
    mean = row_sum(x) / f(n)
    d = x - mean
    rstd = f(1) / np.sqrt(row_sum(d * d) / f(n) + f(eps))
    xh, gh = d * rstd, g * wr
    # one rounding of xh * w + c (a product of 24 and 11 bits is exact in double, and the sum there rounds far below FP32)
    Y = rows((xh.astype(np.float64) * wr + lanes(c[None])).astype(f))
    m1, m2 = row_sum(gh) / f(n), row_sum(gh * xh) / f(n)
    dX = rows(rstd * (gh - m1 - xh * m2))

    def column_sums(t):
        nblocks = -(-b // 32)
        t = np.pad(t, ((0, nblocks * 32 - b), (0, 0))).reshape(nblocks, 32 // waves, waves, n)
        per_wave = t[:, 0]
        for r in range(1, 32 // waves):
            per_wave = per_wave + t[:, r]
        block = per_wave[:, 0]
        for v in range(1, waves):
            block = block + per_wave[:, v]
        seg = np.zeros((16, n), f)
        for k in range(nblocks):
            seg[k % 16] = seg[k % 16] + block[k]
        total = seg[0]
        for k in range(1, 16):
            total = total + seg[k]
        return f(1.0 / np.sqrt(np.float64(b))) * total

    return [a.astype(np.float16) for a in (Y, dX, column_sums(rows(g * xh)), column_sums(rows(g)))]


@pytest.mark.parametrize("b,n,waves", [(1, 16, 16), (77, 496, 16), (600, 1024, 8), (95, 528, 8), (1, 1040, 4), (300, 1552, 4), (64, 2048, 4), (40, 2064, 4),
                                       (70, 4096, 4), (16416, 144, 4), (16416, 528, 4), (8224, 1040, 4)])
def test_rounding_order(b, n, waves):
    """Results are those of the stated FP32 operations, bit for bit: one last place in dw is already 3e-5 of its norm."""
    X, w, c, G = _inputs(b, n, 223 + n, sigma=1.0, shift=0.2)
    with np.errstate(all="ignore"):
        want = _fp32_layer_norm(X, w, c, G, 1e-5, waves)
    for what, a, e in zip(("Y", "dX", "dw", "dc"), _run(X, w, c, G, 1e-5), want):
        assert np.array_equal(a, e), (what, int(np.sum(a != e)))

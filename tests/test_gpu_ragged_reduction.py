"""GPU parity, bit for bit, where the reduction length is no multiple of a pipeline stage (128 FP8 / 64 FP16 elements per
stage, twice that for the wave-split grad_W tile): the last stage is cut by the hardware's range check, on every tile shape and
operand layout, with fewer stages than the ring has slots and with K slices.  Operands are small integers and scales powers of
two, so every partial sum is exact in FP32 and the GPU must equal the oracle whatever the order of the additions."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2303_11257_amd as us
import synth
from gpu_util import DEV, cast_fp8, empty, ptr, stream, to_dev

pytestmark = pytest.mark.gpu


def _operands(shapes, fp8, seed):
    out = []
    for (t, shape), fmt in zip(shapes, (us.E4M3, us.E4M3, us.E5M2)):
        a = synth.small_ints(seed, t, shape)
        out.append(cast_fp8(a, fmt) if fp8 else a)
    return out


# (b, m, n), the product whose reduction is ragged, and a part of the launch record it must show
CASES = [
    ((144, 16, 272), "fwd", "direct:32x32:wk8"), ((144, 48, 272), "fwd", "direct:32x32:wk8"),
    ((1040, 16, 1040), "fwd", "direct:128x128:wk1"), ((1040, 48, 1040), "fwd", "direct:128x128:wk1"),
    ((1040, 112, 1040), "fwd", "direct:128x128:wk1"), ((1040, 144, 1040), "fwd", "direct:128x128:wk1"),
    ((272, 1040, 144), "fwd", None), ((2000, 2064, 1552), "fwd", None),
    ((6144, 176, 4096), "fwd", "direct:256x256"), ((4096, 80, 3072), "fwd", None),
    ((1040, 1040, 16), "dx", "direct:128x128:wk1"), ((1040, 1040, 240), "dx", "direct:128x128:wk1"),
    ((400, 272, 2064), "dx", None), ((4096, 2048, 1040), "dx", None), ((6144, 4096, 208), "dx", "direct:256x256"),
    ((16, 144, 272), "dw", None), ((112, 144, 272), "dw", None), ((1040, 1040, 1040), "dw", ":partial:"),
    ((4112, 400, 272), "dw", ":partial:"), ((2064, 2048, 1536), "dw", "128x128:wk2:st2"), ((272, 4096, 6144), "dw", "direct:256x256"),
    ((2000, 1552, 2064), "fwd", None), ((2000, 1552, 2064), "both", "pair:128x128:wk2:st4"), ((2064, 4096, 1024), "both", "256x128:wk2:st3"), ((4112, 768, 3072), "both", "pair"), ((2096, 3072, 768), "both", "pair"),
]


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])) + c[1])
def test_ragged_reduction(case, fp8):
    (b, m, n), what, record = case
    X, W, G = _operands(((1, (b, m)), (2, (m, n)), (4, (b, n))), fp8, 400 + b + m + n)
    dt = (us.E4M3, us.E4M3, us.E5M2) if fp8 else (us.F16,) * 3
    odt = (O.E4M3, O.E4M3, O.E5M2) if fp8 else (O.F16,) * 3
    tX, tW, tG = to_dev(X), to_dev(W), to_dev(G)
    wsb = us.workspace_bytes(b, m, n)
    ws = torch.full((wsb,), 0x5A, dtype=torch.uint8, device=DEV)
    rows = lambda extent: np.unique(np.concatenate([np.arange(0, extent, max(1, extent // 96)), [extent - 1]]))
    take = lambda t, r: t[torch.as_tensor(r, device=DEV)].cpu().numpy()
    alpha, bx, bw = 2.0 ** -4, 2.0 ** -5, 2.0 ** -6
    rb, rm = rows(b), rows(m)
    if what == "fwd":
        Y = empty((b, n), np.float16)
        us.linear_fwd(ptr(tX), ptr(tW), ptr(Y), b, m, n, dt[0], dt[1], us.F16, alpha, us.EPI_NONE, 0.0, None, None, None, 0, stream())
        rec = us.last_launch()
        assert np.array_equal(take(Y, rb), O.linear_fwd(X[rb], W, alpha, odt[0], odt[1], O.F16)), rec
    else:
        dX = empty((b, m), np.float16) if what != "dw" else None
        dW = empty((m, n), np.float16) if what != "dx" else None
        us.linear_bwd(ptr(tX), ptr(tW), ptr(tG), ptr(dX), ptr(dW), b, m, n, *dt, us.F16, bx, bw, us.EPI_NONE, 0.0, None, None, ptr(ws), wsb,
                      stream())
        rec = us.last_launch()
        if dX is not None:
            assert np.array_equal(take(dX, rb), O.linear_bwd_dx(G[rb], W, bx, odt[2], odt[1], O.F16)), rec
        if dW is not None:
            assert np.array_equal(take(dW, rm), O.linear_bwd_dw(np.ascontiguousarray(X[:, rm]), G, bw, odt[0], odt[2], O.F16)), rec
    assert "direct" in rec or "pair" in rec, rec
    assert record is None or record in rec, rec


def test_a_row_pitch_beyond_32_bit_offsets_takes_the_staged_kernel():
    b, m, n = 16, 1 << 24, 16
    X, W = (np.tile(synth.small_ints(77, t, shape), rep) for t, shape, rep in ((1, (b, 4096), (1, m // 4096)), (2, (4096, n), (m // 4096, 1))))
    X[:, -1] = 1.0                                                  # the tiles are not all alike
    X8, W8 = cast_fp8(X, us.E4M3), cast_fp8(W, us.E4M3)
    tX, tW, Y = to_dev(X8), to_dev(W8), empty((b, n), np.float32)
    us.linear_fwd(ptr(tX), ptr(tW), ptr(Y), b, m, n, us.E4M3, us.E4M3, us.F32, 2.0 ** -12, us.EPI_NONE, 0.0, None, None, None, 0, stream())
    assert "staged" in us.last_launch()
    # integers below 2^24 in absolute value: exact in FP32 and in float64
    ref = (X.astype(np.float32).astype(np.float64) @ W.astype(np.float64)) * 2.0 ** -12
    assert np.max(np.abs(ref)) < 2.0 ** 12 and np.array_equal(Y.cpu().numpy().astype(np.float64), ref)

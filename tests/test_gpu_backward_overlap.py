"""us_linear_bwd with a grad_W that takes the place of the weights or of the saved pre-activation: grad_X reads them first, so the
results are those of the two products alone, bit for bit (small integers: every sum is exact), on shapes of each kind of paired
launch: few tiles, wave-split small tiles, 256 x 128 tiles, and the table-driven activation derivative."""
import numpy as np
import pytest
import torch

import paper_2303_11257_amd as us
import synth
from gpu_util import DEV, cast_fp8, empty, ptr, stream, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("over", ["weights", "preactivation"])
@pytest.mark.parametrize("shape", [(272, 256, 1024), (2000, 1552, 2064), (4096, 768, 3072), (4096, 3072, 768)], ids=lambda s: "x".join(map(str, s)))
def test_grad_w_over_what_grad_x_reads(shape, over, fp8):
    b, m, n = shape
    X, W, G = (synth.small_ints(970 + b, t, s) for t, s in ((1, (b, m)), (2, (m, n)), (4, (b, n))))
    dt = (us.E4M3, us.E4M3, us.E5M2) if fp8 else (us.F16,) * 3
    X, W, G = (cast_fp8(a, f) if fp8 else a for a, f in zip((X, W, G), dt))
    tX, tW, tG, tz = to_dev(X), to_dev(W), to_dev(G), to_dev(synth.normal(971, 11, (b, m)))
    wsb = us.workspace_bytes(b, m, n)
    ws = torch.full((wsb,), 0x5A, dtype=torch.uint8, device=DEV)
    epi = us.EPI_GELU_GRAD if over == "preactivation" else us.EPI_NONE

    def bwd(dX, dW, w=tW, z=tz):
        us.linear_bwd(ptr(tX), ptr(w), ptr(tG), ptr(dX), ptr(dW), b, m, n, *dt, us.F16, 2.0 ** -4, 2.0 ** -4, epi, 0.0,
                      ptr(z) if epi != us.EPI_NONE else None, None, ptr(ws), wsb, stream())
        return us.last_launch()
    dX, dW, dX1, dW1 = empty((b, m), np.float16), empty((m, n), np.float16), empty((b, m), np.float16), empty((m, n), np.float16)
    assert "pair" in bwd(dX, dW)                               # the shape is one that pairs up
    bwd(dX, None), bwd(None, dW)
    src = tW if over == "weights" else tz
    shared = torch.zeros(max(2 * m * n, src.numel() * src.element_size()), dtype=torch.uint8, device=DEV)
    shared[:src.numel() * src.element_size()] = src.view(torch.uint8).flatten()
    assert "pair" not in (bwd(dX1, shared, w=shared) if over == "weights" else bwd(dX1, shared, z=shared))
    assert torch.equal(dX, dX1)
    assert torch.equal(dW.view(torch.uint8).flatten(), shared[:2 * m * n])

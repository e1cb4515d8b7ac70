"""GPU parity, exact, of the large tile on four waves (FP8 products with a 256 x 256 tile for every CU and a long reduction, here about four rounds over 8208): the
three operand layouts with ragged rows, columns and reduction.  Small integers: every sum is exact in FP32 whatever its order,
so sampled rows must equal a float64 product rounded to FP16."""
import pytest
import torch

import paper_2303_11257_amd as us
from gpu_util import DEV, ptr, stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["fwd", "dx", "dw"])
def test_exact(layout):
    M, N, K = 8176, 8016, 8208
    g = torch.Generator(device=DEV).manual_seed(31)
    a, b = (torch.randint(-2, 3, s, generator=g, device=DEV, dtype=torch.int32).to(torch.float16) for s in ((M, K), (N, K)))
    wsb = us.workspace_bytes(M, N, K)
    ws = torch.empty(max(wsb, 16), dtype=torch.uint8, device=DEV)
    C = torch.full((M * N + 64,), 7.0, dtype=torch.float16, device=DEV)

    def codes(x, fmt):
        x, y = x.contiguous(), torch.empty(x.shape, dtype=torch.uint8, device=DEV)
        us.cast_fp8(ptr(x), us.F16, ptr(y), fmt, x.numel(), 1.0, None, stream())
        return y
    s = 2.0 ** -4
    if layout == "fwd":
        A, B = codes(a, us.E4M3), codes(b.t(), us.E4M3)
        us.linear_fwd(ptr(A), ptr(B), ptr(C), M, K, N, us.E4M3, us.E4M3, us.F16, s, us.EPI_NONE, 0.0, None, None, None, 0, stream())
    elif layout == "dx":
        A, B = codes(a, us.E5M2), codes(b, us.E4M3)
        us.linear_bwd(None, ptr(B), ptr(A), ptr(C), None, M, N, K, us.E4M3, us.E4M3, us.E5M2, us.F16, s, s, us.EPI_NONE, 0.0, None, None,
                      None, 0, stream())
    else:
        A, B = codes(a.t(), us.E4M3), codes(b.t(), us.E5M2)
        us.linear_bwd(ptr(A), None, ptr(B), None, ptr(C), K, M, N, us.E4M3, us.E4M3, us.E5M2, us.F16, s, s, us.EPI_NONE, 0.0, None, None,
                      ptr(ws), wsb, stream())
    rec = us.last_launch()
    assert "direct:256x256:wk1:st2:fp8" in rec and rec.endswith(":w4"), rec
    rows = torch.cat([torch.arange(0, M, 97, device=DEV), torch.tensor([M - 1], device=DEV)])
    ref = (a[rows].float().cpu().double() @ b.float().cpu().double().t()) * s
    assert bool((C[M * N:] == 7.0).all())
    assert torch.equal(C[:M * N].view(M, N)[rows].cpu(), ref.to(torch.float16))

"""The matmul epilogues store ragged tiles through buffer resources whose range check drops what lies outside the matrix: every element
of a result is written and nothing in front of it or behind it, for tiles of every shape, FP16 and FP32 results, the activation's
copies and the saved pre-activation; and results with a row pitch beyond the resource's offsets take the register-staged kernel."""
import pytest
import torch

import paper_2303_11257_amd as us
from gpu_util import DEV, ptr, stream

pytestmark = pytest.mark.gpu
GUARD = 1 << 20            # elements on either side of a result: more than the rows that the last tile has beyond it
PATTERN = {torch.float16: 0x7E55, torch.float32: 0x7FC55555, torch.uint8: 0x7F}      # NaNs that no result here is


class Guarded:
    def __init__(self, shape, dtype):
        self.n, self.bits = shape[0] * shape[1], {torch.float16: torch.int16, torch.float32: torch.int32, torch.uint8: torch.uint8}[dtype]
        self.all = torch.full((self.n + 2 * GUARD,), PATTERN[dtype], dtype=self.bits, device=DEV)
        self.pattern = self.all[0].clone()
        self.t = self.all[GUARD:GUARD + self.n].view(dtype).view(shape)

    def check(self):
        inside = self.all[GUARD:GUARD + self.n]
        assert not bool((inside == self.pattern).any())
        assert bool((self.all[:GUARD] == self.pattern).all()) and bool((self.all[GUARD + self.n:] == self.pattern).all())


def _operand(shape, fp8, fmt, seed):
    x = torch.randn(shape, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV).to(torch.float16)
    if not fp8:
        return x, us.F16
    y = torch.empty(shape, dtype=torch.uint8, device=DEV)
    us.cast_fp8(ptr(x), us.F16, ptr(y), fmt, x.numel(), 1.0, None, stream())
    return y, fmt


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("b,m,n", [(4080, 208, 3088), (3856, 1040, 3056), (2000, 1552, 2064), (8176, 1040, 1008), (1040, 1936, 1552), (4096, 768, 3072),
                                   (272, 96, 2224), (80, 4080, 1040)])
def test_ragged_results_stay_inside(b, m, n, fp8):
    (X, xf), (W, wf), (G, gf) = _operand((b, m), fp8, us.E4M3, 1), _operand((m, n), fp8, us.E4M3, 2), _operand((b, n), fp8, us.E5M2, 3)
    z = torch.randn((b, m), device=DEV).to(torch.float16)
    ws = torch.empty(us.workspace_bytes(b, m, n), dtype=torch.uint8, device=DEV)
    w, h, f, c = (ptr(ws), ws.numel(), stream()), torch.float16, torch.float32, torch.uint8
    wide, Y, dX32, dW32 = Guarded((b, n), f), Guarded((b, n), h), Guarded((b, m), f), Guarded((m, n), f)
    us.linear_fwd(ptr(X), ptr(W), ptr(wide.t), b, m, n, xf, wf, us.F32, 0.0, us.EPI_NONE, 0.0, None, None, *w)
    us.linear_fwd(ptr(X), ptr(W), ptr(Y.t), b, m, n, xf, wf, us.F16, 0.0, us.EPI_NONE, 0.0, None, None, *w)
    us.linear_bwd(ptr(X), ptr(W), ptr(G), ptr(dX32.t), ptr(dW32.t), b, m, n, xf, wf, gf, us.F32, 0.0, 0.0, us.EPI_NONE, 0.0, None, None, *w)
    results = [wide, Y, dX32, dW32]
    for act in (0, us.EPI_ACT_RELU):
        Z, H, H8, dZ, dZ8, dW = Guarded((b, n), h), Guarded((b, n), h), Guarded((b, n), c), Guarded((b, m), h), Guarded((b, m), c), Guarded((m, n), h)
        us.linear_fwd(ptr(X), ptr(W), ptr(Z.t), b, m, n, xf, wf, us.F16, 0.0, us.EPI_GELU | act, 0.0, ptr(H.t), ptr(H8.t), *w)
        us.linear_bwd(ptr(X), ptr(W), ptr(G), ptr(dZ.t), ptr(dW.t), b, m, n, xf, wf, gf, us.F16, 0.0, 0.0, us.EPI_GELU_GRAD | act, 0.0, ptr(z),
                      ptr(dZ8.t), *w)
        results += [Z, H, H8, dZ, dZ8, dW]
        assert torch.equal(Z.t, Y.t)
    dR = Guarded((b, m), h)
    us.linear_bwd(None, ptr(W), ptr(G), ptr(dR.t), None, b, m, n, xf, wf, gf, us.F16, 0.0, 0.0, us.EPI_RESIDUAL, 0.6, ptr(z), None, *w)
    for r in results + [dR]:
        r.check()


def test_grad_x_with_a_long_result_pitch():
    """2^25 columns: the operands' pitches are short, the result's is not (64 MB a row).  Small integers, exact."""
    b, m, n = 16, 1 << 25, 16
    G = torch.randint(-2, 3, (b, n), device=DEV).to(torch.float16)
    W = torch.randint(-2, 3, (m, n), device=DEV, dtype=torch.int8).to(torch.float16)
    dX = torch.empty((b, m), dtype=torch.float16, device=DEV)
    us.linear_bwd(None, ptr(W), ptr(G), ptr(dX), None, b, m, n, *(us.F16,) * 4, 0.25, 0.0, us.EPI_NONE, 0.0, None, None, None, 0, stream())
    assert "staged" in us.last_launch()
    assert torch.equal(dX, (G.float() @ W.float().t() * 0.25).to(torch.float16))


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_longest_result_pitch_of_the_direct_kernels(dtype):
    """2^25 - 16 columns: 32 FP32 rows are 2048 bytes short of the 4 GB that a resource can span, and offsets run up to there.  48 rows are one
    whole strip and half of one; the rows that the tile has beyond them are part of the buffer here and must keep their pattern.  Small
    integers, exact."""
    b, m, n = 48, (1 << 25) - 16, 16
    G = torch.randint(-2, 3, (b, n), device=DEV).to(torch.float16)
    W = torch.randint(-2, 3, (m, n), device=DEV, dtype=torch.int8).to(torch.float16)
    bits = torch.int16 if dtype == torch.float16 else torch.int32
    pattern, rows = PATTERN[dtype], 256 + 64             # the largest tile, and as much as the farthest offset of a lane beyond its last strip
    all_ = torch.full((rows * m + GUARD,), pattern, dtype=bits, device=DEV)
    dX = all_[GUARD:GUARD + b * m].view(dtype).view(b, m)
    us.linear_bwd(None, ptr(W), ptr(G), ptr(dX), None, b, m, n, us.F16, us.F16, us.F16, us.F32 if dtype == torch.float32 else us.F16, 0.25, 0.0, us.EPI_NONE, 0.0,
                  None, None, None, 0, stream())
    assert us.last_launch().startswith("direct:256x256"), us.last_launch()
    for i in range(0, b, 8):
        assert torch.equal(dX[i:i + 8], (G[i:i + 8].float() @ W.float().t() * 0.25).to(dtype)), i
    assert bool((all_[:GUARD] == pattern).all())
    for part in all_[GUARD + b * m:].split(1 << 30):
        assert bool((part == pattern).all())

"""GPU parity, exact, of products whose reduction has no more stages than the ring and of those just beyond, on the tiles that have a form of their own for them:
128 x 128 (FP16), 256 x 192, and 256 x 256 (FP8), ragged in every dimension.  Small integers: sums stay below 2^24, so the FP32 product of torch is exact too."""
import pytest
import torch

import paper_2303_11257_amd as us
from gpu_util import DEV, ptr, stream
from test_gpu_one_round_large_tile import _dx, _fwd, _operand

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epi", ["plain", "bias", "relu", "residual"])
@pytest.mark.parametrize("K", [16, 64, 80, 128, 144])
def test_forward_small_tile(K, epi):
    assert "direct:128x128:wk1:st2:f16" in _fwd(2032, 2576, K, False, epi)


@pytest.mark.parametrize("K", [16, 128, 144])
def test_forward_wide_tile(K):
    assert "direct:256x192:wk1" in _fwd(4080, 3072, K, False, "plain")
    assert "direct:256x192:wk1" in _fwd(4080, 3072, K, False, "gelu")


@pytest.mark.parametrize("epi", ["plain", "relu", "gelu", "residual"])
@pytest.mark.parametrize("K", [16, 128, 144, 256, 272])
def test_forward_large_tile(K, epi):
    assert "direct:256x256:wk1:st2:fp8" in _fwd(4080, 3600, K, True, epi)


@pytest.mark.parametrize("epi", ["plain", "relu"])
@pytest.mark.parametrize("M,N,K,fp8", [(2032, 2576, 16, False), (2032, 2576, 128, False), (2032, 2576, 144, False), (4080, 3600, 256, True)])
def test_grad_x(M, N, K, fp8, epi):
    assert ("direct:256x256:wk1:st2:fp8" if fp8 else "direct:128x128:wk1:st2:f16") in _dx(M, N, K, fp8, epi)


@pytest.mark.parametrize("M,N,K,fp8", [(2032, 2576, k, False) for k in (16, 128, 144, 192, 208)] + [(4080, 3600, k, True) for k in (16, 256, 272)])
def test_grad_w(M, N, K, fp8):
    (X, Xo, xd), (G, Go, gd) = _operand((K, M), fp8, us.E4M3, 5), _operand((K, N), fp8, us.E5M2, 6)
    for dt, out in ((us.F16, torch.float16), (us.F32, torch.float32)):
        dW = torch.full((M * N + 64,), 7.0, dtype=out, device=DEV)
        us.linear_bwd(ptr(Xo), None, ptr(Go), None, ptr(dW), K, M, N, xd, us.E4M3 if fp8 else us.F16, gd, dt, 0.0, 2.0 ** -5, us.EPI_NONE, 0.0, None, None, None, 0, stream())
        rec = us.last_launch()
        assert ("direct:256x256:wk1:st2:fp8" if fp8 else "direct:128x128:wk1:st2:f16") in rec, rec
        want = (X.float().t().contiguous() @ G.float() * 2.0 ** -5).to(out)
        assert torch.equal(dW[:M * N].view(M, N), want) and bool((dW[M * N:] == 7.0).all()), rec

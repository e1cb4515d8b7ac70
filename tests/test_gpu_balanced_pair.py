"""GPU parity, exact, of a layer's two backward products on four-wave 128 x 128 tiles in one launch where the tiles do not all run from the
start or one product has few of them: ragged edges, more tiles than slots, each epilogue, both operand types, and the layers just beside."""
import pytest

from test_gpu_two_per_cu_pair import PAIR, _bwd

pytestmark = pytest.mark.gpu
ACT = [(2048, 2048, 512), (1568, 2624, 656), (528, 2528, 1264),        # up to seven eighths of the slots
       (2800, 4112, 416), (7536, 4112, 464)]                          # many tiles with a short reduction of grad_X
ACT_FP8 = [(5104, 2064, 1008), (4128, 3088, 1264)]                     # ... in bytes: with FP8 operands only
REST = [(2064, 1680, 912), (1552, 1808, 784), (640, 2192, 1392)]       # no derivative: up to eleven sixteenths of the slots


@pytest.mark.parametrize("b,m,n,epi,fp8", [(*s, "relu", f) for s in ACT for f in (False, True)] + [(*s, "relu", True) for s in ACT_FP8] +
                         [(*s, e, f) for s in REST for e in ("plain", "residual") for f in (False, True)])
def test_pair_is_exact(b, m, n, epi, fp8):
    p, e = "fp8" if fp8 else "f16", {"plain": "store", "relu": "act_grad", "residual": "residual"}[epi]
    assert _bwd(b, m, n, fp8, epi) == PAIR.format(p=p, e=e)


# Layers on either side of a limit, which are in bytes of reduction (FP16: half as many values)
@pytest.mark.parametrize("fp8,b,m,n,epi,taken", [
    (False, 6976, 416, 3280, "relu", False), (True, 6112, 416, 3280, "relu", True), (True, 6144, 416, 3280, "relu", False),   # few grad_W tiles, long reduction
    (False, 1712, 848, 6272, "relu", False), (True, 1712, 848, 6128, "relu", True), (True, 1712, 848, 6144, "relu", False),   # few grad_X tiles, long reduction
    (False, 9280, 3488, 400, "relu", False), (True, 18176, 1792, 896, "relu", False),                                       # few grad_W tiles next to many rounds
    (False, 2432, 3072, 752, "relu", True), (False, 2432, 3072, 768, "relu", False),            # instead of 256 x 128 tiles: below 1536 bytes
    (True, 4992, 2048, 1520, "relu", True), (True, 4992, 2048, 1536, "relu", False), (False, 4992, 2048, 1024, "relu", False),
    (True, 4128, 3088, 1264, "relu", True), (True, 4128, 3088, 1280, "relu", False),            # more tiles than slots: below 1280 bytes
    (False, 2800, 2048, 512, "plain", False), (True, 2800, 2048, 512, "plain", False)])         # no derivative, more than eleven sixteenths of the slots
def test_beside_the_window(fp8, b, m, n, epi, taken):
    pair = PAIR.format(p="fp8" if fp8 else "f16", e="act_grad" if epi == "relu" else "store")
    assert (_bwd(b, m, n, fp8, epi) == pair) == taken

"""GPU parity of the fused attention rows (us_attention.hip) at the edges of its kernels: row lengths around every limit where the
query block or the lanes per row change, rows that end inside a 32-key step or a staged chunk, query blocks with rows beyond the
sequence, head sizes that fill or do not fill the matrix instruction's steps, few and many heads (the two workgroup orders),
and the shapes beside the window, which take the separate kernels."""
import numpy as np
import pytest
import torch

import paper_2303_11257_amd as us
from gpu_util import DEV, ptr, stream
from test_gpu_attention import Attn, check_heads

pytestmark = pytest.mark.gpu

SHAPES = [(2, 16, 16), (1, 48, 32), (40, 112, 64), (3, 128, 80), (33, 144, 48), (2, 240, 128), (1, 256, 64), (2, 272, 32), (1, 496, 96),
          (34, 512, 64), (1, 528, 64), (2, 528, 128), (1, 1008, 16), (1, 1024, 112), (2, 1040, 64), (1, 1232, 128), (1, 2048, 32),
          (1, 2064, 64), (1, 128, 144),
          # at least 256 heads and 65 to 128 keys: scores in registers (one and two 64-key chunks, ragged head sizes), and beside it
          (256, 64, 64), (255, 128, 64), (256, 80, 64), (259, 96, 32), (256, 112, 48), (256, 128, 16), (300, 128, 64), (256, 128, 80),
          (256, 112, 128),
          # score tensors of 64 MB and more leave with non-temporal stores; dV and dK on 256-row tiles
          (130, 512, 64), (513, 256, 32)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_against_the_oracle(shape):
    heads, s, d = shape
    check_heads(Attn(heads, s, d, 500 + s + d), sorted({0, heads // 2, heads - 1}))


@pytest.mark.parametrize("heads", [2, 256])
def test_special_values_stay_in_their_rows(heads):
    """A NaN or +inf score makes its whole row of P (and of O) NaN and no other; results beyond the tensors are untouched."""
    s, d = 80, 48
    g = torch.Generator(device="cpu").manual_seed(5)
    Q, K, V = (torch.randn((heads, s, d), generator=g).to(torch.float16).to(DEV) for _ in range(3))
    Q[0, 3, 0] = float("nan")
    Q[1, 79, :] = 0.0
    Q[1, 79, 0] = float("inf")
    K[1, :, 0] = 1.0
    n = heads * s * s
    A, P = (torch.full((n + 64,), 7.0, dtype=torch.float16, device=DEV) for _ in range(2))
    O = torch.full((heads * s * d + 64,), 7.0, dtype=torch.float16, device=DEV)
    us.attention_fwd(ptr(Q), ptr(K), ptr(V), ptr(A), ptr(P), ptr(O), heads, s, d, stream())
    torch.cuda.synchronize()
    assert bool((A[n:] == 7.0).all()) and bool((P[n:] == 7.0).all()) and bool((O[heads * s * d:] == 7.0).all())
    bad = np.zeros((heads, s), bool)
    bad[0, 3] = bad[1, 79] = True
    p, o = P[:n].view(heads, s, s).isnan().cpu().numpy(), O[:heads * s * d].view(heads, s, d).isnan().cpu().numpy()
    assert np.array_equal(p.all(-1), bad) and np.array_equal(p.any(-1), bad)
    assert np.array_equal(o.all(-1), bad) and np.array_equal(o.any(-1), bad)


def test_results_over_inputs_no_longer_needed():
    """A result that takes the place of an array which the separate steps have finished with by then is the same result."""
    heads, s, d = 3, 128, 128                                  # [heads, s, s] and [heads, s, d] are the same size
    g = torch.Generator(device="cpu").manual_seed(6)
    new = lambda: torch.empty((heads, s, s), dtype=torch.float16, device=DEV)
    Q, K, V, dO = (torch.randn((heads, s, d), generator=g).to(torch.float16).to(DEV) for _ in range(4))
    A, P, O, dP, dA, dQ, dK, dV = (new() for _ in range(8))
    st = stream()

    def fwd(q, k, v, a, p, o):
        us.attention_fwd(ptr(q), ptr(k), ptr(v), ptr(a), ptr(p), ptr(o), heads, s, d, st)

    def bwd(v, a, p, do, dp, da, dq):
        us.attention_bwd(ptr(Q), ptr(K), ptr(v), ptr(a), ptr(p), ptr(do), ptr(dp), ptr(da), ptr(dq), ptr(dK), ptr(dV), heads, s, d, st)
        return dK.clone(), dV.clone()
    fwd(Q, K, V, A, P, O)
    kv = bwd(V, A, P, dO, dP, dA, dQ)
    near = lambda x, y: bool(((x.float() - y.float()).norm() <= 4e-4 * y.float().norm()).item())   # FP16 results, sums in another order
    for over in ("o_k", "o_q", "p_a", "p_k"):
        q, k, a, p, o = Q.clone(), K.clone(), new(), new(), new()
        p = a if over == "p_a" else k if over == "p_k" else p
        o = k if over == "o_k" else q if over == "o_q" else o
        fwd(q, k, V, a, p, o)
        assert near(p, P) and near(o, O), over
    for over in ("dq_v", "dq_do", "dq_a", "da_v", "dp_p", "da_dp", "da_a"):
        v, do, a, p, dp, da, dq = V.clone(), dO.clone(), A.clone(), P.clone(), new(), new(), new()
        dq = {"dq_v": v, "dq_do": do, "dq_a": a}.get(over, dq)
        dp = p if over == "dp_p" else dp
        da = {"da_v": v, "da_dp": dp, "da_a": a}.get(over, da)
        kv2 = bwd(v, a, p, do, dp, da, dq)
        assert near(dq, dQ) and near(da, dA) and near(kv2[0], kv[0]) and near(kv2[1], kv[1]), over


@pytest.mark.parametrize("heads", [3, 256])
@pytest.mark.parametrize("over", ["dk_do", "dk_p", "dk_k", "dk_v", "dk_a", "dk_dp", "dv_dk", "dv_dp"])
def test_key_and_value_gradients_over_other_arrays(over, heads):
    """The separate steps make dV first and dK last.  A dK that takes the place of an array with no reader left by then is the same
    result; a dV in the place of a later result leaves that result as it is."""
    s = d = 128                                                # [heads, s, s] and [heads, s, d] are the same size
    g = torch.Generator(device="cpu").manual_seed(7)
    new = lambda: torch.empty((heads, s, s), dtype=torch.float16, device=DEV)
    Q, K, V, dO = (torch.randn((heads, s, d), generator=g).to(torch.float16).to(DEV) for _ in range(4))
    A, P, O = (new() for _ in range(3))
    us.attention_fwd(ptr(Q), ptr(K), ptr(V), ptr(A), ptr(P), ptr(O), heads, s, d, stream())

    def bwd(k, v, a, p, do, dp, da, dq, dk, dv):
        us.attention_bwd(ptr(Q), ptr(k), ptr(v), ptr(a), ptr(p), ptr(do), ptr(dp), ptr(da), ptr(dq), ptr(dk), ptr(dv), heads, s, d, stream())
    dP, dA, dQ, dK, dV = (new() for _ in range(5))
    bwd(K, V, A, P, dO, dP, dA, dQ, dK, dV)
    k, v, a, p, do, dp, da, dq, dk, dv = K.clone(), V.clone(), A.clone(), P.clone(), dO.clone(), *(new() for _ in range(5))
    dk = {"dk_do": do, "dk_p": p, "dk_k": k, "dk_v": v, "dk_a": a, "dk_dp": dp}.get(over, dk)
    dv = {"dv_dk": dk, "dv_dp": dp}.get(over, dv)
    bwd(k, v, a, p, do, dp, da, dq, dk, dv)
    near = lambda x, y: bool(((x.float() - y.float()).norm() <= 4e-4 * y.float().norm()).item())   # FP16 results, sums in another order
    assert near(dk, dK) and near(dq, dQ) and near(da, dA)
    assert over.startswith("dv") or near(dv, dV)
    assert over == "dk_dp" or near(dp, dP)


@pytest.mark.parametrize("heads,s,d,rows,pair", [(2, 512, 64, "rows:64x512:wk1", "pair:128x64:"), (256, 128, 128, "rows:128x128:wk1", "pair:128x128:"),
                                                 (1, 2048, 32, "rows:16x2048:wk4", "pair:128x64:"), (1, 2064, 64, None, None)])
def test_launch_record(heads, s, d, rows, pair):
    """One entry per launch of the forward call, and the rows and the two products behind them for the backward call."""
    t = lambda *shape: torch.zeros(shape, dtype=torch.float16, device=DEV)
    Q, K, V, O, dO, dQ, dK, dV = (t(heads, s, d) for _ in range(8))
    A, P, dP, dA = (t(heads, s, s) for _ in range(4))
    us.attention_fwd(ptr(Q), ptr(K), ptr(V), ptr(A), ptr(P), ptr(O), heads, s, d, stream())
    fwd = us.last_launch().split(" + ")
    us.attention_bwd(ptr(Q), ptr(K), ptr(V), ptr(A), ptr(P), ptr(dO), ptr(dP), ptr(dA), ptr(dQ), ptr(dK), ptr(dV), heads, s, d, stream())
    bwd = us.last_launch().split(" + ")
    if rows is None:
        assert [e.split(":")[0] for e in fwd] == ["direct"] * 2 and [e.split(":")[0] for e in bwd] == ["direct"] * 4
        return
    assert len(fwd) == 1 and fwd[0].startswith(rows) and fwd[0].endswith(":f16:NT:softmax:s1")
    assert len(bwd) == 3 and bwd[0].startswith(rows) and bwd[0].endswith(":f16:NT:softmax_grad:s1")
    assert all(e.startswith(pair) and e.endswith(":f16:TN:store:s1") for e in bwd[1:])


@pytest.mark.parametrize("heads,s,d,fwd,bwd", [(4, 1536, 128, False, True), (2, 1536, 128, True, True), (10, 1040, 128, False, False), (9, 1024, 128, False, True),
                                               (12, 1040, 96, False, True), (34, 1248, 80, False, False), (8, 2048, 64, False, True), (16, 2048, 48, False, False),
                                               (7, 1600, 48, True, True), (128, 512, 128, False, False), (50, 512, 128, False, True),
                                               (16, 512, 128, True, True), (50, 512, 112, True, True), (6, 1536, 112, False, True)])
def test_one_kernel_only_where_it_is_faster(heads, s, d, fwd, bwd):
    """Both sides of the lines beyond which many long rows or wide heads take the separate kernels, forward and backward apart."""
    a = Attn(heads, s, d, 900 + s + d)
    us.attention_fwd(*(ptr(a.t[n]) for n in ("Q", "K", "V", "A", "P", "O")), heads, s, d, stream())
    assert us.last_launch().startswith("rows") == fwd, us.last_launch()
    us.attention_bwd(*(ptr(a.t[n]) for n in ("Q", "K", "V", "A", "P", "dO", "dP", "dA", "dQ", "dK", "dV")), heads, s, d, stream())
    assert us.last_launch().startswith("rows") == bwd, us.last_launch()
    check_heads(a, [heads - 1])


@pytest.mark.parametrize("heads,s,d", [(2, 112, 64), (256, 128, 64), (2, 512, 64), (1, 1008, 80), (1, 1232, 96), (2, 2064, 64)])
def test_a_probability_on_one_key_has_no_gradient(heads, s, d):
    """Every row of P is s on one key and zero elsewhere: p (dP - sum p dP) is zero, exactly, whatever the size of the scores and of dP."""
    g = torch.Generator(device="cpu").manual_seed(8)
    K, V, dO = (torch.randn((heads, s, d), generator=g).to(torch.float16).to(DEV) for _ in range(3))
    perm = torch.randperm(s, generator=g).to(DEV)
    Q = (64.0 * K[:, perm]).contiguous()
    t = {n: torch.empty((heads, s, s if n in ("A", "P", "dP", "dA") else d), dtype=torch.float16, device=DEV)
         for n in ("A", "P", "O", "dP", "dA", "dQ", "dK", "dV")}
    us.attention_fwd(ptr(Q), ptr(K), ptr(V), ptr(t["A"]), ptr(t["P"]), ptr(t["O"]), heads, s, d, stream())
    us.attention_bwd(ptr(Q), ptr(K), ptr(V), ptr(t["A"]), ptr(t["P"]), ptr(dO), ptr(t["dP"]), ptr(t["dA"]), ptr(t["dQ"]), ptr(t["dK"]), ptr(t["dV"]),
                     heads, s, d, stream())
    top = t["A"].float().topk(2, -1).values
    alone = top[..., 0] - top[..., 1] > 110.0                   # every other exponential is zero in FP32
    assert float(alone.float().mean()) > 0.99
    assert bool((t["P"][alone].float().sum(-1) == s).all()) and not bool(t["dA"][alone].any())

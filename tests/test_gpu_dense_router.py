"""The router's adjoint without renormalisation (every expert's gradient is nonzero): the dense router term of the
input-gradient hand-back and the weight gradient of more than 32 experts, where token tiles (16), expert steps (16, 64)
and 32-token chunks end, against fp64 sums of the same inputs."""
import numpy as np
import pytest
import torch

from paper_2506_02965_amd import pcmoe as P
from gpu_util import log

pytestmark = pytest.mark.gpu

CASES = [  # T, d, E, k, shared, dtype
    (1, 128, 9, 2, 0, "bf16"), (15, 256, 16, 3, 1, "bf16"), (17, 128, 33, 8, 2, "f32"), (33, 384, 50, 5, 3, "bf16"),
    (64, 128, 64, 1, 0, "f32"), (129, 640, 65, 4, 0, "bf16"), (1030, 256, 256, 8, 0, "bf16"), (16500, 256, 64, 2, 0, "bf16"),
    (8300, 256, 130, 4, 0, "f32"), (33000, 128, 33, 1, 0, "bf16"),
    (515, 128, 255, 6, 1, "f32"), (2050, 2048, 9, 2, 0, "bf16"), (2049, 2048, 11, 1, 1, "bf16"), (2050, 2048, 9, 3, 0, "bf16"),
    (2047, 2048, 9, 2, 0, "bf16"), (1023, 2048, 250, 8, 0, "bf16"), (100, 1024, 100, 4, 0, "bf16"),
]


def _inputs(T, d, E, k, S, dtype, seed=5):
    g = torch.Generator().manual_seed(seed)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    n = lambda *s: torch.randn(*s, generator=g)
    x, wr, dxp = n(T, d).to(dt), (n(E, d) * d ** -0.5).to(dt), n(T * k + S * T, d).to(dt)
    idx = torch.stack([torch.randperm(E, generator=g)[:k] for _ in range(T)]).int()
    s2r = torch.randperm(T * k, generator=g).int()
    return x, wr, dxp, idx, s2r, n(T, E), n(T, k)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "T{}_d{}_E{}_k{}_S{}_{}".format(*c))
def test_dense_router_adjoint(case):
    T, d, E, k, S, dtype = case
    log(f"[dense router] {case}")
    x, wr, dxp, idx, s2r, logits, dgate = _inputs(*case)
    desc = P.make_desc(T, d, 128, E, k, 0, E, S, False, dtype)
    dev = lambda t: t.cuda().contiguous()
    dl, dwr = torch.empty(T, E, device="cuda"), torch.empty(E, d, device="cuda")
    dx = torch.empty(T, d, device="cuda", dtype=x.dtype)
    ws = torch.empty(max(P.moe_workspace_size(desc, P.MOE_WS_ROUTE_BWD), 1), dtype=torch.uint8, device="cuda")
    topk_w = torch.softmax(logits.double(), 1).gather(1, idx.long()).float()
    P.moe_route_bwd(desc, dev(x), dev(logits), dev(idx), dev(topk_w), dev(dgate), dl, dwr, ws, ws.numel())
    P.moe_permute_bwd(desc, dev(dxp), dev(s2r), dl, dev(wr), dx)
    torch.cuda.synchronize()
    p = torch.softmax(logits.double(), 1)
    gg = torch.zeros(T, E, dtype=torch.float64).scatter_(1, idx.long(), dgate.double())
    ref_dl = p * (gg - (p * gg).sum(1, keepdim=True))
    got_dl = dl.cpu().double()
    # fp32 exp, division and one 64-lane sum: a few ulp of the largest entry
    assert (got_dl - ref_dl).abs().max() <= 1e-5 * ref_dl.abs().max()
    # the products take the gradients the kernel was given
    ref_dw = got_dl.t() @ x.double()
    assert (dwr.cpu().double() - ref_dw).abs().max() <= 1e-5 * ref_dw.abs().max()   # fp32 sums over T
    rows = dxp.double()
    ref_dx = rows[s2r.long()].view(T, k, d).sum(1) + got_dl @ wr.double()
    for s in range(S):
        ref_dx = ref_dx + rows[T * k + s * T:T * k + (s + 1) * T]
    tol = 2 ** -8 if dtype == "bf16" else 1e-5   # one rounding to bf16 of the fp32 sum
    assert (dx.cpu().double() - ref_dx).abs().max() <= tol * ref_dx.abs().max()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_zero_gradient_skips_infinite_weights(dtype):
    """An expert whose gradient is zero contributes nothing even where its router row is infinite or NaN."""
    T, d, E, k = 40, 256, 20, 2
    log(f"[dense router] infinite row {dtype}")
    x, wr, dxp, idx, s2r, _, _ = _inputs(T, d, E, k, 0, dtype)
    dl = torch.randn(T, E)
    dl[:, 7] = 0.0
    dl[3, 11] = 0.0
    ref = dxp.double()[s2r.long()].view(T, k, d).sum(1) + dl.double() @ wr.double()
    wr[7] = float("inf")
    wr[7, ::2] = float("nan")
    desc = P.make_desc(T, d, 128, E, k, 0, E, 0, False, dtype)
    dx = torch.empty(T, d, device="cuda", dtype=x.dtype)
    P.moe_permute_bwd(desc, dxp.cuda(), s2r.cuda(), dl.cuda(), wr.cuda(), dx)
    torch.cuda.synchronize()
    tol = 2 ** -8 if dtype == "bf16" else 1e-5
    assert (dx.cpu().double() - ref).abs().max() <= tol * ref.abs().max()
    assert np.isfinite(dx.float().cpu().numpy()).all()


@pytest.mark.parametrize("T,d,E,tokens", [(8192, 2048, 256, 256), (16384, 2048, 64, 128), (8192, 2048, 64, 64)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_router_gradient_error(T, d, E, tokens, dtype):
    """The error of dW_router's fp32 sums against fp64 of the same gradients is that of accumulators over `tokens` tokens.
    A sum of n independent terms, rounded after each, is off by u c sqrt(n / 2) of its size: the j-th partial sum is
    sqrt(j / n) of it, and a rounding is off by c = 0.425 units u = 2^-24 of the value in the mean (mantissas spread
    over their logarithm). The chunks are then added 16 ways and the 16 sums in turn. 10% are left for the spread."""
    log(f"[dW_router error] T={T} d={d} E={E} {dtype}")
    k = 2
    gen = torch.Generator(device="cuda").manual_seed(3)
    n = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    x, logits, dgate = n(T, d).to(torch.bfloat16 if dtype == "bf16" else torch.float32), n(T, E), n(T, k)
    topk_w, idx = torch.topk(torch.softmax(logits, 1), k)
    desc = P.make_desc(T, d, 128, E, k, 0, E, 0, False, dtype)
    dl, dwr = torch.empty(T, E, device="cuda"), torch.empty(E, d, device="cuda")
    ws = torch.empty(max(P.moe_workspace_size(desc, P.MOE_WS_ROUTE_BWD), 1), dtype=torch.uint8, device="cuda")
    P.moe_route_bwd(desc, x, logits, idx.int().contiguous(), topk_w.contiguous(), dgate, dl, dwr, ws, ws.numel())
    ref = dl.double().t().contiguous() @ x.double()
    err = float((dwr.double() - ref).norm() / ref.norm())
    steps = tokens + T / tokens / 16 + 16
    bound = 1.1 * 2 ** -24 * 0.425 * (steps / 2) ** 0.5
    log(f"[dW_router error] {err:.3e}, bound {bound:.3e}")
    assert err <= bound

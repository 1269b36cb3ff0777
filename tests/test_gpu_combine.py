"""The combine's adjoint on both sides of the size from which it reads its rows non-temporally (128 MiB of routed rows):
output-row gradients bit-exact, gate gradients against fp64."""
import pytest
import torch

from paper_2506_02965_amd import pcmoe as P
from gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,k,dtype", [(4096, 2, "bf16"), (2048, 2, "f32"), (4096, 8, "bf16")])
def test_combine_bwd_large_rows(d, k, dtype):
    """The same tokens in a batch just below the line and at it: equal bits; some tokens' rows are absent (-1)."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    T = (128 << 20) // (k * d * (2 if dtype == "bf16" else 4))
    log(f"[combine_bwd] d={d} k={k} {dtype} T={T}")
    gen = torch.Generator(device="cuda").manual_seed(3)
    dy, yp = (torch.randn(n, d, device="cuda", generator=gen).to(dt) for n in (T, T * k))
    gw = torch.rand(T, k, device="cuda", generator=gen)
    s2r = torch.randperm(T * k, device="cuda", generator=gen).int()
    s2r[5], s2r[T * k - 1] = -1, -1
    out = []
    for t in (T - 1, T):
        dyp = torch.full((T * k, d), 7.0, device="cuda", dtype=dt)
        dgate = torch.full((T, k), 7.0, device="cuda")
        P.moe_combine_bwd(P.make_desc(t, d, 128, 8, k, dtype=dtype), dy, yp, s2r, gw, dyp, dgate)
        torch.cuda.synchronize()
        out.append((dyp, dgate))
    slots = torch.arange(T * k, device="cuda")
    for t, (dyp, dgate) in zip((T - 1, T), out):
        live = slots[(s2r >= 0) & (slots < t * k)]
        rows, tok = s2r[live].long(), live // k
        want = torch.full_like(dyp, 7.0)
        want[rows] = (gw.reshape(-1)[live, None] * dy[tok].float()).to(dt)
        assert torch.equal(dyp, want)
        dot = torch.zeros(T * k, device="cuda", dtype=torch.float64)
        mag = torch.zeros_like(dot)
        for a in range(0, live.numel(), 4096):
            s = slice(a, a + 4096)
            p = dy[tok[s]].double() * yp[rows[s]].double()
            dot[live[s]], mag[live[s]] = p.sum(1), p.abs().sum(1)
        got = dgate.reshape(-1)[:t * k].double()
        # d fp32 products, each added with one rounding: in every order below d * 2^-24 of the sum of magnitudes
        assert ((got - dot[:t * k]).abs() <= d * 2.0 ** -24 * mag[:t * k]).all()
        assert torch.equal(dgate[t:], torch.full_like(dgate[t:], 7.0))
    assert torch.equal(out[0][1][:T - 1], out[1][1][:T - 1])

"""The router forward at the edges of its dispatch (1, 4, 16 or 32 tokens per workgroup, 16 to 256 expert columns)
against fp64 scores: selection bit-exact, scores within one ulp of fp32, gate weights within 1e-5 (the bar of the
parity tests)."""
import pytest
import torch

from paper_2506_02965_amd import pcmoe as P
from gpu_util import check_logits, log

pytestmark = pytest.mark.gpu


def route(T, d, E, k, dtype, renorm=True, edit=None, bias=None, seed=5):
    gen = torch.Generator().manual_seed(seed)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn(T, d, generator=gen).to(dt)
    w = (torch.randn(E, d, generator=gen) * d ** -0.5).to(dt)
    if edit:
        edit(x, w)
    desc = P.make_desc(T, d, 128, E, k, renormalize=renorm, dtype=dtype)
    logits = torch.full((T, E), 7.0, device="cuda")
    idx = torch.full((T, k), -3, dtype=torch.int32, device="cuda")
    gw = torch.full((T, k), -3.0, device="cuda")
    P.moe_route(desc, x.cuda(), w.cuda(), None if bias is None else bias.cuda(), 1 if bias is None else bias.shape[0],
                logits, idx, gw)
    torch.cuda.synchronize()
    s = x.double() @ w.double().t()
    if bias is not None:
        s = s + bias.double().repeat_interleave(T // bias.shape[0], 0)
    return s, logits.cpu(), idx.cpu(), gw.cpu()


def check(s, logits, idx, gw, k, renorm):
    check_logits(logits, s.float().numpy())
    ref = torch.sort(logits, dim=1, descending=True, stable=True).indices[:, :k]   # ties to the lower index
    assert torch.equal(idx.long(), ref)
    p = torch.softmax(s, 1).gather(1, ref)
    p = p / p.sum(1, keepdim=True) if renorm else p
    assert float((gw.double() - p).abs().max() / p.abs().max()) <= 1e-5


CASES = [(1, 128, 4, 2), (3, 256, 16, 1), (256, 128, 17, 8), (257, 384, 16, 3), (255, 2048, 64, 6), (1024, 128, 65, 4),
         (1025, 640, 64, 6), (1030, 128, 33, 2), (4096, 128, 129, 8), (4097, 256, 256, 8), (4100, 128, 32, 2),
         (5000, 128, 8, 2), (300, 256, 256, 8), (2000, 256, 200, 8), (7, 512, 100, 8), (4099, 128, 64, 6),
         (4098, 256, 128, 4), (8200, 128, 17, 2), (8195, 256, 40, 6), (8193, 128, 100, 4), (8199, 128, 256, 8),
         (12400, 128, 32, 2), (12300, 128, 64, 6)]


@pytest.mark.parametrize("T,d,E,k", CASES)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_route_dispatch_edges(T, d, E, k, dtype):
    renorm = (T + E) % 2 == 0
    bias = torch.randn(1, E, generator=torch.Generator().manual_seed(T))
    log(f"[router] T={T} d={d} E={E} k={k} {dtype} renormalize={renorm}")
    check(*route(T, d, E, k, dtype, renorm, bias=bias), k, renorm)


@pytest.mark.parametrize("T", [5, 500, 2000, 5000])
def test_route_special_scores(T):
    """Equal scores, -0 beside +0, -inf scores and a NaN expert, in each token tiling."""
    d, E, k = 128, 70, 8

    def edit(x, w):
        w[3] = w[66]
        w[10] = 0
        w[11] = 0
        w[40, 5] = float("nan")

    bias = torch.zeros(1, E)
    bias[0, 20] = float("-inf")
    s, logits, idx, gw = route(T, d, E, k, "bf16", edit=edit, bias=bias)
    assert torch.isnan(logits[:, 40]).all() and torch.isneginf(logits[:, 20]).all()
    keep = [e for e in range(E) if e != 40]   # the NaN expert is never selected
    ref = torch.sort(logits[:, keep], dim=1, descending=True, stable=True).indices[:, :k]
    assert torch.equal(idx.long(), torch.tensor(keep)[ref])
    # fewer selectable experts than k - 1: -inf scores are taken in index order
    bias = torch.full((1, E), float("-inf"))
    bias[0, 69], bias[0, 64] = 0.0, 1e4
    s, logits, idx, gw = route(T, d, E, 4, "bf16", bias=bias)
    assert torch.equal(idx, torch.tensor([64, 69, 0, 1], dtype=torch.int32).expand(T, 4))
    assert torch.equal(gw, torch.tensor([1.0, 0.0, 0.0, 0.0]).expand(T, 4))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_route_batch_size(dtype):
    """The same tokens in batches of different size (1, 4, 16 and 32 tokens per workgroup). Where fp64 holds every sum
    exactly (inputs on a grid: here multiples of 2^-6 of at most 8 significant bits) the scores are the same bits in
    each; else they lie within one ulp of fp32, and calls of the same size give the same bits."""
    d, E, k, sizes = 640, 64, 6, (1, 300, 2000, 5000)
    log(f"[router] batch size {dtype}")
    gen = torch.Generator().manual_seed(8)
    all_x, all_w = torch.randn(max(sizes), d, generator=gen), torch.randn(E, d, generator=gen) * d ** -0.5
    grid = lambda t: (t * 64).round().clamp(-127, 127) / 64

    def run(T, on_grid):
        def same_tokens(x, w):
            x.copy_(grid(all_x[:T]) if on_grid else all_x[:T])
            w.copy_(grid(all_w) if on_grid else all_w)
        return route(T, d, E, k, dtype, edit=same_tokens)

    s, logits, idx, gw = run(max(sizes), True)
    assert torch.equal(logits, s.float())   # the exact sums, rounded once
    for T in sizes[:-1]:
        _, lg, ix, g = run(T, True)
        assert torch.equal(lg, logits[:T]) and torch.equal(ix, idx[:T]) and torch.equal(g, gw[:T]), T
    for T in sizes:
        s, lg, ix, g = run(T, False)
        check_logits(lg, s.float().numpy())
        assert all(torch.equal(a, b) for a, b in zip((lg, ix, g), run(T, False)[1:])), T

"""The bf16 expert GEMMs of few rows per expert (weights streamed into registers) where their row chunks (16, 32, 64 and
128 rows), column blocks and 64-deep K steps end, and the scan that finds a workgroup's group among up to 64, 128 and
more groups. The backward reads the tile plan that the gate/up launch wrote."""
import numpy as np
import pytest
import torch

from paper_2506_02965_amd import pcmoe as P
from paper_2506_02965_amd.layer import LayerWeights, MoELayer
from paper_2506_02965_amd.synth import LayerConfig, make_inputs
from gpu_util import check_full, log, run_gpu

pytestmark = pytest.mark.gpu


def _fill(E, edges, total):
    """Rows per expert: the edges, zeros between, and the rest spread over the remaining experts."""
    left = E - len(edges)
    rest = total - sum(edges)
    assert rest >= 0
    return list(edges) + [rest // left + (1 if i < rest % left else 0) for i in range(left)]


def _case(T, d, f, E, edges, seed, **kw):
    cfg = LayerConfig("st", T=T, d=d, f=f, E=E, k=2, bias="party", parties=T, seed=seed, **kw)
    return cfg, _fill(E, edges, 2 * T)


CASES = {
    # expected rows per group <= 8: single wavefronts (16-row chunks), one or two column blocks each
    "split": _case(48, 256, 384, 16, [0, 1, 15, 16, 17, 33, 0], 71),
    "split_k_remainder_shared": _case(24, 128, 128, 12, [16, 0, 17], 72, n_shared=2),
    "split_66_groups": _case(130, 128, 256, 64, [0, 16, 1, 40], 73, n_shared=2),
    # <= 24: 32-row chunks
    "rows32": _case(130, 256, 384, 16, [0, 1, 31, 32, 33, 65], 74),
    "rows32_130_groups": _case(700, 128, 128, 130, [0, 32, 33], 75),
    # <= 50: 64-row chunks, one and two column blocks per wavefront of the down projection
    "rows64": _case(300, 256, 640, 16, [0, 63, 64, 65, 129, 1], 76, n_shared=1),
    "rows64_wide": _case(640, 1024, 128, 40, [0, 63, 64, 65, 130], 77),
    # few workgroups and a long K: 8 steps in flight, 32- and 64-row chunks (the latter in place of 128)
    "rows32_deep": _case(60, 256, 1152, 8, [0, 31, 33, 1], 83),
    "rows64_deep": _case(150, 256, 1024, 8, [0, 63, 64, 65, 1], 84),
    "rows64_few": _case(300, 256, 1408, 8, [0, 63, 129, 1], 85),
    # <= 100 (and up to 200 where the tile grid is small): 128-row chunks
    "rows128": _case(515, 384, 256, 8, [0, 127, 128, 129, 257, 1], 78),
    "rows128_narrow": _case(400, 1024, 128, 12, [0, 127, 128, 129, 1], 86),
    "rows128_wide": _case(1100, 1024, 128, 40, [0, 127, 128, 129, 258], 79),
    # ... and two column blocks per wavefront of the down projection
    "rows128_two_blocks": _case(600, 2048, 128, 8, [0, 127, 128, 129, 258, 1], 94),
    # more than 128 groups: a lane of the group scan counts eight of them
    "split_130_groups": _case(300, 128, 128, 130, [0, 16, 17, 40, 1], 95),
    "split_258_groups": _case(64, 128, 256, 256, [0, 17, 33, 1], 96, n_shared=2),
    # one column block of a few rows; two blocks in the down projection; its 32-row chunks where many experts are active
    "one_block": _case(16, 256, 384, 16, [0, 16, 1, 3], 97),
    "down_two_blocks": _case(96, 2048, 128, 24, [0, 16, 17, 31, 1], 98),
    "down_rows32_many": _case(40, 2048, 1024, 16, [0, 16, 17, 33, 1], 99),
}


# a long d_ff beside few columns: the streamed dX, 16- and 32-row chunks, several groups of more than one chunk
CASES.update({
    "dx16": _case(24, 256, 2816, 4, [0, 16, 17], 87),
    "dx32": _case(65, 128, 2944, 4, [65, 33, 0], 88, n_shared=1),
    "dx_mid": _case(150, 384, 2816, 6, [31, 32, 0, 129], 89),
    "dx_skew": _case(150, 256, 2816, 6, [100, 70, 33, 31, 0], 90),
})


def forced(inp, counts):
    T = inp.cfg.T
    assert sum(counts) == 2 * T and max(counts) <= T
    slots = np.repeat(np.arange(len(counts)), counts)  # a token's two slots lie T apart: different experts
    inp.logit_bias[:] = -1e4
    t = np.arange(T)
    inp.logit_bias[t, slots[:T]] = 2e4
    inp.logit_bias[t, slots[T:]] = 1e4


@pytest.mark.parametrize("name", list(CASES))
def test_stream_edges(name):
    cfg, counts = CASES[name]
    log(f"[stream] {name}")
    inp = make_inputs(cfg, with_dy=True)
    forced(inp, counts)
    layer, _ = run_gpu(cfg, inp)
    assert np.array_equal(layer.counts.cpu().numpy(), counts)
    errs = check_full(cfg, inp, layer)
    log(f"[stream] {name}: " + " ".join(f"{k}={v:.2e}" for k, v in errs.items()))


def test_stream_shard_one_token():
    """A shard that hosts a quarter of the experts, and a single token (most groups empty)."""
    for cfg in (LayerConfig("st1", T=130, d=256, f=128, E=32, k=4, local_begin=8, local_count=8, n_shared=1,
                            router_backward=False, seed=81),
                LayerConfig("st2", T=1, d=256, f=384, E=64, k=6, n_shared=2, seed=82)):
        inp = make_inputs(cfg, with_dy=True)
        layer, _ = run_gpu(cfg, inp)
        check_full(cfg, inp, layer)


@pytest.mark.parametrize("name", ["split", "rows32", "rows64", "rows128", "dx_mid", "dx_skew"])
def test_non_finite_weights_stay_in_their_rows(name):
    """A NaN in one expert's W_gate and an infinity in another's W_down reach the rows of these experts alone: every
    other row, padded ones of the same chunk included, has the bits of a run without them."""
    cfg, counts = CASES[name]
    log(f"[stream] non-finite weights: {name}")
    inp = make_inputs(cfg, with_dy=True)
    forced(inp, counts)
    clean, _ = run_gpu(cfg, inp)
    bad, inf = [e for e, c in enumerate(counts) if c > 1][:2]
    inp.w_gate[bad, 5] = np.nan
    inp.w_down[inf, 7] = np.inf
    layer, _ = run_gpu(cfg, inp)
    off = np.concatenate([[0], np.cumsum(counts)])
    rows = lambda e: slice(off[e], off[e + 1])
    assert torch.equal(layer.offsets, clean.offsets) and torch.equal(layer.slot_to_row, clean.slot_to_row)
    y, y0, dx, dx0 = layer.y_perm, clean.y_perm, layer.dx_perm, clean.dx_perm
    assert bool(torch.isnan(y[rows(bad)]).all()) and bool(torch.isnan(dx[rows(bad)]).all())
    assert not bool(torch.isfinite(y[rows(inf), 7]).any())
    other = [c for c in range(cfg.d) if c != 7]
    assert torch.equal(y[rows(inf)][:, other], y0[rows(inf)][:, other])
    keep = [e for e in range(cfg.E) if e not in (bad, inf)]
    for e in keep:
        assert torch.equal(y[rows(e)], y0[rows(e)]) and torch.equal(dx[rows(e)], dx0[rows(e)]), e
        assert torch.equal(layer.dw_gate[e], clean.dw_gate[e]) and torch.equal(layer.dw_down[e], clean.dw_down[e]), e
    shared = slice(2 * cfg.T, 2 * cfg.T + cfg.n_shared * cfg.T)
    assert torch.equal(y[shared], y0[shared]) and torch.equal(dx[shared], dx0[shared])


@pytest.mark.parametrize("d,f,E,k,S", [(256, 384, 16, 2, 1), (512, 1408, 40, 4, 0), (4096, 1024, 8, 2, 0)])
def test_forward_bits_do_not_depend_on_the_batch(d, f, E, k, S):
    """A token's expert outputs are the same bits whatever kernel its batch's size selects: single wavefronts, 32-, 64-
    and 128-row chunks and the LDS tiles sum over K in one order."""
    log(f"[stream] bits over batch sizes, d={d} f={f} E={E}")
    sizes = (1, 7, 24, 70, 200, 500, 4096)
    gen = torch.Generator(device="cuda").manual_seed(4)
    new = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=gen) * std).to(torch.bfloat16)
    G = E + S
    x, w_router = new(max(sizes), d), new(E, d, std=d ** -0.5)
    wg, wu, wd = new(G, f, d, std=d ** -0.5), new(G, f, d, std=d ** -0.5), new(G, d, f, std=f ** -0.5)
    out = {}
    for T in sizes:
        layer = MoELayer(LayerConfig("bits", T=T, d=d, f=f, E=E, k=k, n_shared=S, backward=False))
        layer.forward(LayerWeights(x[:T].contiguous(), w_router, None, 1, wg, wu, wd))
        torch.cuda.synchronize()
        rows = layer.slot_to_row.long().view(T, k)
        shared = T * k + T * torch.arange(S, device="cuda")[None] + torch.arange(T, device="cuda")[:, None]
        out[T] = (layer.topk_idx.clone(), layer.y_perm[torch.cat([rows, shared], 1)].clone())
    ref_idx, ref = out[max(sizes)]
    for T, (idx, y) in out.items():
        assert torch.equal(idx, ref_idx[:T]), T
        assert torch.equal(y, ref[:T]), T


def launches(T, d, f, E, k, local=None, S=0, backward=False):
    """Names of the launches of a layer's expert passes."""
    cfg = LayerConfig("rt", T=T, d=d, f=f, E=E, k=k, local_count=local, n_shared=S, router_backward=False,
                      backward=backward)
    gen = torch.Generator(device="cuda").manual_seed(1)
    new = lambda *s: torch.randn(*s, device="cuda", dtype=torch.bfloat16, generator=gen) * 0.02
    G = cfg.n_groups
    w = LayerWeights(new(T, d), new(E, d), None, 1, new(G, f, d), new(G, f, d), new(G, d, f), new(T, d))
    layer = MoELayer(cfg)
    P.moe_kernel_timing(True)
    layer.forward(w)
    if backward:
        layer.backward(w)
    torch.cuda.synchronize()
    names = set(P.moe_kernel_timing_report())
    P.moe_kernel_timing(False)
    return names


@pytest.mark.parametrize("T,d,f,E,k,local,tiles", [
    (777, 1024, 2816, 16, 2, None, False), (792, 2048, 1408, 16, 2, None, True), (640, 2048, 2816, 16, 2, None, True),
    (400, 2048, 5632, 16, 2, None, True), (200, 2048, 5632, 16, 2, None, False), (1280, 2048, 1408, 64, 1, None, True),
    (192, 2048, 1408, 64, 4, 16, False), (320, 2048, 1408, 64, 4, 16, True), (384, 1024, 2816, 32, 2, 8, True),
])
def test_gate_up_route(T, d, f, E, k, local, tiles):
    """Gate/up goes to the LDS tiles (which need the tile plan launched first) at row counts where streamed chunks are
    slower once the routing is skewed, though they are not on uniform rows."""
    log(f"[stream] route of gate/up, T={T} d={d} f={f} E={E} k={k} local={local}")
    assert ("ffn_plan" in launches(T, d, f, E, k, local)) == tiles


@pytest.mark.parametrize("T,d,f,E,k,local,streamed", [
    (400, 1024, 2816, 16, 2, None, True), (1024, 1024, 2816, 16, 2, None, False), (48, 4096, 2816, 4, 2, None, False),
    (60, 4096, 5632, 2, 1, None, True), (288, 768, 1408, 16, 2, None, False), (500, 1024, 2816, 32, 4, 8, True),
    (1000, 1024, 2816, 32, 4, 8, False),
])
def test_dx_route(T, d, f, E, k, local, streamed):
    """dX is streamed only where that beats the launch it otherwise shares with dW_gate, dW_up."""
    log(f"[stream] route of dX, T={T} d={d} f={f} E={E} k={k} local={local}")
    names = launches(T, d, f, E, k, local, backward=True)
    assert ("gemm_bwd_dx" in names) == streamed and ("gemm_bwd_dx+wgrad_gate_up" in names) != streamed


def _no_tokens(inp):
    inp.logit_bias[0, 0] = -1e4


@pytest.mark.parametrize("name", ["shard_one_group", "shard_without_rows", "two_groups"])
def test_streamed_dx_beside_pipelined_weight_gradient(name):
    """d_model = 4096: dX streamed, and dW_gate, dW_up in a launch of their own on the pipelined tile, over one chunk of
    rows, several, and none."""
    kw = dict(d=4096, E=2, k=1)
    cfg, edit = {
        "shard_one_group": (LayerConfig("dp1", T=130, f=2048, local_count=1, router_backward=False, seed=91, **kw), None),
        "shard_without_rows": (LayerConfig("dp2", T=60, f=2048, local_count=1, router_backward=False, bias="forced_empty",
                                           seed=92, **kw), _no_tokens),
        "two_groups": (LayerConfig("dp3", T=44, f=5632, seed=93, **kw), None),
    }[name]
    log(f"[stream] dX at d_model 4096: {name}")
    inp = make_inputs(cfg, with_dy=True)
    if edit:
        edit(inp)
    P.moe_kernel_timing(True)
    layer, _ = run_gpu(cfg, inp)
    names = set(P.moe_kernel_timing_report())
    P.moe_kernel_timing(False)
    assert {"gemm_bwd_dx", "gemm_wgrad_gate_up"} <= names
    errs = check_full(cfg, inp, layer)
    log(f"[stream] {name}: " + " ".join(f"{k}={v:.2e}" for k, v in errs.items()))

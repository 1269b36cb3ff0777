"""The fp32 expert GEMMs where their 64 x 64 tiles and 32-deep K-tiles end: row counts of 0, 1, 63, 64, 65 and more,
weight-gradient K loops with a remainder, the smallest d_model and d_ff, shards and shared experts."""
import numpy as np
import pytest

from paper_2506_02965_amd.synth import LayerConfig, make_inputs
from gpu_util import check_full, log, run_gpu

pytestmark = pytest.mark.gpu

COUNTS = [0, 1, 63, 64, 65, 97, 110]   # rows per expert: 2 T slots, none above T = 200


def forced(inp):
    T = inp.cfg.T
    slots = np.repeat(np.arange(len(COUNTS)), COUNTS)
    assert slots.size == 2 * T
    inp.logit_bias[:] = -1e4
    t = np.arange(T)
    inp.logit_bias[t, slots[:T]] = 2e4
    inp.logit_bias[t, slots[T:]] = 1e4


CASES = {
    "edges_small": (LayerConfig("fe1", T=200, d=128, f=128, E=7, k=2, bias="party", parties=200, dtype="f32", seed=61), forced),
    "edges_d384_shared": (LayerConfig("fe2", T=200, d=384, f=256, E=7, k=2, bias="party", parties=200, n_shared=2,
                                      dtype="f32", seed=62), forced),
    "one_token": (LayerConfig("fe3", T=1, d=256, f=384, E=4, k=2, n_shared=1, dtype="f32", seed=63), None),
    "shard": (LayerConfig("fe4", T=515, d=256, f=128, E=32, k=4, local_begin=8, local_count=8, router_backward=False,
                          dtype="f32", seed=64), None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_f32_tiles(name):
    cfg, edit = CASES[name]
    log(f"[f32] {name}")
    inp = make_inputs(cfg, with_dy=True)
    if edit:
        edit(inp)
    layer, _ = run_gpu(cfg, inp)
    errs = check_full(cfg, inp, layer)
    log(f"[f32] {name}: " + " ".join(f"{k}={v:.2e}" for k, v in errs.items()))

"""The dispatch at the slot counts where it changes from one launch to three and where a wavefront's slots end, on full
layers and shards: maps, counts and gathered rows against a stable sort."""
import numpy as np
import pytest
import torch

from paper_2506_02965_amd import pcmoe as P
from gpu_util import log

pytestmark = pytest.mark.gpu

CASES = [  # T, k, E, first hosted expert, hosted experts, d
    (1, 1, 1, 0, 1, 128), (1, 6, 64, 0, 64, 2048), (63, 1, 8, 0, 8, 128), (65, 1, 8, 2, 3, 128), (1024, 1, 4, 0, 4, 128),
    (1025, 1, 4, 0, 4, 128), (171, 6, 64, 16, 16, 640), (512, 8, 256, 0, 256, 256), (683, 6, 33, 0, 33, 128),
    (4097, 1, 32, 0, 32, 128), (4096, 2, 32, 31, 1, 128), (4096, 2, 33, 0, 33, 128), (2731, 3, 16, 0, 16, 4096),
    (8193, 1, 5, 0, 5, 128), (40, 8, 8, 7, 1, 128),
]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "T{}_k{}_E{}_from{}_host{}_d{}".format(*c))
def test_permute(case, dtype):
    T, k, E, lb, lc, d = case
    log(f"[permute] {case} {dtype}")
    rng = np.random.default_rng(T + E)
    idx = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    if T > 100:
        idx[:T // 2, 0] = idx[0, 0]   # one expert with half the tokens (it may repeat in a row: only the order counts)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn(T, d, generator=torch.Generator().manual_seed(1)).to(dt)
    desc = P.make_desc(T, d, 128, E, k, lb, lc, 0, True, dtype)
    new = lambda *s, t=torch.int32: torch.full(s, -7, dtype=t, device="cuda")
    counts, offsets, r2s, s2r, xp = new(lc), new(lc + 1), new(T * k), new(T * k), new(T * k, d, t=dt)
    ws = torch.empty(max(P.moe_workspace_size(desc, P.MOE_WS_PERMUTE), 1), dtype=torch.uint8, device="cuda")
    P.moe_permute(desc, torch.from_numpy(idx).cuda(), x.cuda(), counts, offsets, r2s, s2r, xp, ws, ws.numel())
    torch.cuda.synchronize()
    local = idx.reshape(-1) - lb
    hosted = np.nonzero((local >= 0) & (local < lc))[0]
    rows = hosted[np.argsort(local[hosted], kind="stable")]
    n = len(rows)
    ref_counts = np.bincount(local[hosted], minlength=lc)
    assert np.array_equal(counts.cpu().numpy(), ref_counts)
    assert np.array_equal(offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(ref_counts)]))
    assert np.array_equal(r2s.cpu().numpy(), np.concatenate([rows, np.full(T * k - n, -1)]))
    ref_s2r = np.full(T * k, -1)
    ref_s2r[rows] = np.arange(n)
    assert np.array_equal(s2r.cpu().numpy(), ref_s2r)
    assert torch.equal(xp[:n].cpu(), x[torch.from_numpy(rows // k)])
    assert bool((xp[n:] == -7).all())   # rows past the hosted ones are not written

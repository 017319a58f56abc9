"""Class rows at every width that takes another kernel or another form of the row loads (K a multiple of 4 or not, rows
16-byte aligned or not), logits and probabilities, against the oracle; rows that are not finite stay in their voxels."""
import numpy as np
import pytest
import torch

from _gpu_util import assert_stats_equal, compare_maps, cuda, extract_np, make_pair
from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 3, 4, 8, 9, 16, 17, 20, 24, 25, 32, 33, 64])
@pytest.mark.parametrize("kind", [sv.IN_LOGIT_F32, sv.IN_PROB_F32])
def test_rows(K, kind):
    fr = synth.room_frame(seed=K, width=41, height=23, f=30.0, cx=20.5, cy=11.5)
    n = len(fr["points"])
    rng = np.random.default_rng(K)
    rows = rng.standard_normal((n, K)).astype(np.float32) * 3
    if kind == sv.IN_PROB_F32:
        rows = np.abs(rows)
    g, o = make_pair(0.1, 0.3, 0.0, 100.0, sv.SEM_CLOSED, K, 0, 1 << 10, 1 << 16)
    h = sv.Map(0.1, 0.3, 0.0, 100.0, sv.SEM_CLOSED, K, 0, 0, 1 << 10, 1 << 16)
    p = cuda(fr["points"])
    off = torch.empty(n * K + 1, device="cuda")[1:].view(n, K)  # 4-byte aligned
    off.copy_(cuda(rows))
    for _ in range(2):
        g.integrate(p, fr["pose"], cuda(rows), kind)
        assert_stats_equal(g.stats(), o.integrate(fr["points"], fr["pose"], rows, kind))
        h.integrate(p, fr["pose"], off, kind)
    x, y = extract_np(g), extract_np(h)
    compare_maps(x, o.extract(), 0.3, sv.SEM_CLOSED, K)
    for k in x:
        assert np.array_equal(x[k], y[k]), k
    # a row with NaN and one with an infinity: D and W unchanged by them, the other voxels' counts too
    bad = rows.copy()
    bad[n // 3, K // 2] = np.nan
    bad[n // 2, 0] = np.inf
    for m, r in ((g, bad), (h, rows)):
        m.reset()
        m.integrate(p, fr["pose"], cuda(r), kind)
    x, y = extract_np(g), extract_np(h)
    assert np.array_equal(x["D"], y["D"]) and np.array_equal(x["W"], y["W"])
    hit = ~np.isfinite(x["sem"]).all(axis=1)
    assert 0 < hit.sum() < 100
    assert np.array_equal(x["sem"][~hit], y["sem"][~hit])
    g.close()
    h.close()

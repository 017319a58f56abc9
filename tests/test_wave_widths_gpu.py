"""The general wave combine at the row lengths where its components per lane change (64, 128, 256), with voxels of one
to several hundred observations, against the batched launch (which takes 16 components per lane for every length), bit
for bit, and the oracle's counts and geometry."""
import numpy as np
import pytest
import torch

from _gpu_util import assert_stats_equal, cuda, make_pair
from paper_2512_12945_amd import slimvdb as sv

pytestmark = pytest.mark.gpu

WIDTHS = [(sv.SEM_OPEN, 0, L, k) for L, k in ((1, "f32"), (63, "f32"), (64, "bf16"), (65, "f32"), (100, "bf16"), (127, "f32"),
                                               (129, "f32"), (255, "bf16"), (257, "f32"), (1000, "f32"))]
WIDTHS += [(sv.SEM_CLOSED, K, 0, k) for K, k in ((33, "label"), (33, "prob"), (64, "logit"), (65, "prob"), (128, "label"),
                                                 (129, "prob"), (256, "label"), (256, "prob"))]


@pytest.mark.parametrize("mode,K,L,kind", WIDTHS)
def test_widths(mode, K, L, kind):
    n = 700
    rng = np.random.default_rng(K * 2000 + L)
    p = np.stack([1.0 + rng.normal(0.0, 0.01, n), rng.uniform(-0.5, 0.5, n), rng.uniform(-0.3, 0.3, n)], axis=1)
    p[:300, 1:] = rng.uniform(0.01, 0.04, (300, 2))  # one voxel's width
    p = p.astype(np.float32)
    if kind == "label":
        s, k = rng.integers(0, K, n).astype(np.int32), sv.IN_LABEL_I32
    elif K:
        s, k = np.abs(rng.standard_normal((n, K))).astype(np.float32), sv.IN_PROB_F32 if kind == "prob" else sv.IN_LOGIT_F32
    else:
        s, k = rng.standard_normal((n, L)).astype(np.float32), sv.IN_EMB_F32
        if kind == "bf16":
            s, k = (s.view(np.uint32) >> 16).astype(np.uint16), sv.IN_EMB_BF16
    g, o = make_pair(0.05, 0.15, 0.0, 10.0, mode, K, L, 1 << 10, 1 << 16)
    b = sv.Map(0.05, 0.15, 0.0, 10.0, mode, K, L, 0, 1 << 10, 1 << 16)
    b.set_launch_shape(batch_mode=2)
    pt, st = cuda(p), cuda(s)
    for _ in range(2):
        g.integrate(pt, np.eye(4), st, k)
        sv.integrate_batched([b], [dict(points=pt, pose=np.eye(4), sem=st, kind=k)])
        assert_stats_equal(g.stats(), o.integrate(p, np.eye(4), s, k))
    x, y, ox = g.extract(), b.extract(), o.extract()
    for name in x:
        assert torch.equal(x[name].view(torch.int32), y[name].view(torch.int32)), name
    assert np.array_equal(x["keys"].cpu().numpy(), ox["keys"])
    assert np.array_equal(x["W"].cpu().numpy().astype(np.float64), ox["W"]) and float(x["W"].max()) > 256
    assert np.all(np.abs(x["D"].cpu().numpy() - ox["D"]) <= 1e-5 * np.maximum(np.abs(ox["D"]), 0.15))
    g.close()
    b.close()

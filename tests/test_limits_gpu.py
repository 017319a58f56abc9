"""The widest truncation a map accepts: 6 voxel sizes, also where their binary32 product rounds upwards and a ray may
visit 43 cells instead of 40; one unit in the last place above is refused."""
import numpy as np
import pytest
import torch

import oracle
from _gpu_util import assert_stats_equal, compare_maps, cuda, extract_np, integrate_both, make_pair
from oracle import loss as ol
from paper_2512_12945_amd import slimvdb as sv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vs", [0.1, 0.125, 0.0700000152])
def test_widest_band(vs):
    vs = np.float32(vs)
    tau = np.float32(6.0) * vs
    K, n = 4, 700
    with pytest.raises(sv.SlimError):
        sv.Map(float(vs), float(np.nextafter(tau, np.float32(9.0))), 0.0, 100.0, sv.SEM_CLOSED, K)
    rng = np.random.default_rng(3)
    d = rng.standard_normal((n, 3))
    d[::3] = rng.choice([-1.0, 1.0], (len(d[::3]), 3)) + rng.normal(0.0, 1e-3, (len(d[::3]), 3))  # diagonals: the most cells
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    r = rng.uniform(2.0, 3.0, n).astype(np.float32)
    logits = rng.standard_normal((n, K)).astype(np.float32)
    g, o = make_pair(float(vs), float(tau), 0.0, 100.0, sv.SEM_CLOSED, K, 0, 1 << 12, 1 << 19)
    pts = ol.rays_to_points(r, d)
    gs, os_ = integrate_both(g, o, pts, np.eye(4), logits, sv.IN_LOGIT_F32)
    assert_stats_equal(gs, os_)
    ex = o.extract()
    compare_maps(extract_np(g), ex, tau, sv.SEM_CLOSED, K)
    y = rng.integers(0, K, len(ex["W"])).astype(np.int32)
    samples = ((ex["keys"][::5] + 0.5) * np.float64(vs)).astype(np.float32)
    lo = ol.map_loss(ex, y, samples, float(vs))
    g.loss(cuda(ex["keys"]), cuda(y), cuda(samples))
    gl, gr = torch.empty(n, K, device="cuda"), torch.empty(n, device="cuda")
    g.backward_rays(cuda(r), cuda(d), np.eye(4), cuda(logits), gl, gr)
    want_l, want_r, _ = ol.frame_gradients(o, dict(ranges=r, dirs=d, pose=np.eye(4), logits=logits), ex, lo)
    for got, want in ((gl, want_l), (gr, want_r)):
        got, want = got.cpu().numpy().astype(np.float64), np.asarray(want)
        assert np.all(np.abs(got - want) <= 1e-5 * (np.abs(want) + np.abs(want).max())), np.abs(got - want).max()
    g.close()

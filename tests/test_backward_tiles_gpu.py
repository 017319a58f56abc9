"""Loss and gradients at the edges of the backward's vectors (K + 1 adjoints in 1, 2 or 3 vectors of 16 per ray) and
workgroups (64 rays), with logits that are only 4-byte aligned, rejected rays, voxels that the loss does not list and
rays that were not integrated, against the oracle's FP64 gradient (1e-5 of |g| + max |g|, as the full workload's test)."""
import numpy as np
import pytest
import torch

import oracle
from _gpu_util import cuda
from oracle import loss as ol
from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth

pytestmark = pytest.mark.gpu

VS, TAU = 0.1, 0.6  # the longest band: 6 voxels either side


def rays(n, K, seed):
    fr = synth.room_frame(seed=seed, width=40, height=30, f=30.0, cx=20.0, cy=15.0)
    p = fr["points"].astype(np.float64)
    r = np.linalg.norm(p, axis=1)
    pick = np.random.default_rng(seed).permutation(len(r))[:n]
    d = (p / r[:, None])[pick].astype(np.float32)
    r = r[pick].astype(np.float32)
    if n > 10:
        r[n // 2] = np.nan  # a rejected ray
    logits = (np.random.default_rng(seed + 1).standard_normal((n, K)) * 2).astype(np.float32)
    return dict(ranges=r, dirs=d, pose=fr["pose"], logits=logits)


@pytest.mark.parametrize("K,n", [(1, 63), (3, 1), (4, 64), (11, 65), (15, 300), (16, 129), (20, 257), (31, 64), (32, 1000)])
@pytest.mark.parametrize("aligned", [True, False])
def test_gradients(K, n, aligned):
    fr = rays(n, K, K * 7 + n)
    om = oracle.OracleMap(VS, TAU, 0.0, 50.0, oracle.SEM_CLOSED, K)
    om.integrate(ol.rays_to_points(fr["ranges"], fr["dirs"]), fr["pose"], fr["logits"], oracle.IN_LOGIT_F32)
    ex = om.extract()
    M = len(ex["W"])
    rng = np.random.default_rng(n)
    y = rng.integers(-1, K + 1, M).astype(np.int32)
    samples = ((ex["keys"][rng.integers(0, M, 300)] + 0.5) * np.float64(np.float32(VS))).astype(np.float32)
    listed = np.arange(M) if n < 100 else np.flatnonzero(rng.random(M) < 0.7)
    lo = ol.map_loss(ex, y, samples, VS)
    g = sv.Map(VS, TAU, 0.0, 50.0, sv.SEM_CLOSED, K, 0, 0, 1 << 12, 1 << 18)
    r, d = cuda(fr["ranges"]), cuda(fr["dirs"])
    buf, out = torch.empty(n * K + 1, device="cuda"), torch.full((n * K + 2,), 5.0, device="cuda")
    o = 0 if aligned else 1
    lg, gl = buf[o:o + n * K].view(n, K), out[o:o + n * K].view(n, K)
    lg.copy_(cuda(fr["logits"]))
    gr = torch.empty(n, device="cuda")
    scale = torch.full((1,), 0.5, device="cuda")
    g.integrate_rays(r, d, fr["pose"], lg, sv.IN_LOGIT_F32)
    # a first loss of other labels leaves rows behind, the second is the one that counts
    keys, sm = cuda(ex["keys"]), cuda(samples)
    g.loss(keys, cuda(((y + 2) % K).astype(np.int32)), sm)
    if len(listed) == M:
        loss = g.loss(keys, cuda(y), sm)
        assert abs(float(loss[0]) - lo["loss"]) <= 1e-5 * abs(lo["loss"])
        g.backward_rays(r, d, fr["pose"], lg, gl, gr, grad_scale=scale)
        want_l, want_r, _ = ol.frame_gradients(om, fr, ex, lo)
    else:
        # the voxels that are not listed carry zero adjoints; the means are over those listed
        g.loss(keys[cuda(listed)].contiguous(), cuda(y[listed]), sm)
        g.backward_rays(r, d, fr["pose"], lg, gl, gr, grad_scale=scale)
        on = np.zeros(M, bool)
        on[listed] = True
        lo = dict(lo, adj_c=np.where(on[:, None], lo["adj_c"] * M / len(listed), 0.0), adj_D=np.where(on, lo["adj_D"], 0.0))
        want_l, want_r, _ = ol.frame_gradients(om, fr, ex, lo)
    for got, want in ((gl, want_l), (gr, want_r)):
        got, want = got.cpu().numpy().astype(np.float64), 0.5 * np.asarray(want)
        assert np.all(np.abs(got - want) <= 1e-5 * (np.abs(want) + np.abs(want).max())), np.abs(got - want).max()
    assert out[n * K + o] == 5.0 and (aligned or out[0] == 5.0)
    # rays that were not integrated: leaves, pages and voxels that are not there add nothing
    far = r.clone()
    far += 3.0
    g.backward_rays(far, d, fr["pose"], lg, gl, gr)
    assert torch.isfinite(gl).all() and torch.isfinite(gr).all()
    g.close()

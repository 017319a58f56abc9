"""Backward of rays that were not integrated: what their walks meet outside the map adds exactly nothing -- no leaf at all,
leaves or pages that are not there, and voxels of the map in between, against the oracle's adjoints gathered along the
walk (1e-5 of |g| + max |g|, as the full workload's test)."""
import numpy as np
import pytest
import torch

import oracle
from _gpu_util import cuda
from oracle import loss as ol
from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth

pytestmark = pytest.mark.gpu

VS, TAU = 0.1, 0.3


@pytest.mark.parametrize("K", [3, 20, 32])
def test_rays_off_the_map(K):
    fr = synth.room_frame(seed=3, width=40, height=30, f=30.0, cx=20.0, cy=15.0)
    p = fr["points"].astype(np.float64)
    r = np.linalg.norm(p, axis=1)
    dirs, r = (p / r[:, None]).astype(np.float32), r.astype(np.float32)
    n = len(r)
    rng = np.random.default_rng(K)
    logits = (rng.standard_normal((n, K)) * 2).astype(np.float32)
    om = oracle.OracleMap(VS, TAU, 0.0, 50.0, oracle.SEM_CLOSED, K)
    om.integrate(ol.rays_to_points(r, dirs), fr["pose"], logits, oracle.IN_LOGIT_F32)
    ex = om.extract()
    M = len(ex["W"])
    y = rng.integers(0, K, M).astype(np.int32)
    samples = ((ex["keys"][::2] + 0.5) * np.float64(np.float32(VS))).astype(np.float32)
    lo = ol.map_loss(ex, y, samples, VS)
    g = sv.Map(VS, TAU, 0.0, 50.0, sv.SEM_CLOSED, K, 0, 0, 1 << 12, 1 << 18)
    d, lg = cuda(dirs), cuda(logits)
    g.integrate_rays(cuda(r), d, fr["pose"], lg, sv.IN_LOGIT_F32)
    g.loss(cuda(ex["keys"]), cuda(y), cuda(samples))

    def back(ranges):
        gl, gr = torch.full((n, K), 7.0, device="cuda"), torch.full((n,), 7.0, device="cuda")
        g.backward_rays(cuda(ranges), d, fr["pose"], lg, gl, gr)
        return gl.cpu().numpy().astype(np.float64), gr.cpu().numpy().astype(np.float64)

    for away in (20.0, 3.0):  # past every leaf, and past the walls by more than the band
        gl, gr = back(r + np.float32(away))
        assert np.all(gl == 0.0) and np.all(gr == 0.0)
    # half of the band inside: the map of these rays alone names the voxels that their walks meet
    near = (r + np.float32(0.25)).astype(np.float32)
    gl, gr = back(near)
    o2 = oracle.OracleMap(VS, TAU, 0.0, 50.0, oracle.SEM_CLOSED, K)
    o2.integrate(ol.rays_to_points(near, dirs), fr["pose"], logits, oracle.IN_LOGIT_F32)
    e2 = o2.extract()
    at = {tuple(k): i for i, k in enumerate(ex["keys"])}
    row = np.array([at.get(tuple(k), -1) for k in e2["keys"]])
    on = row >= 0
    assert 0.1 < on.mean() < 0.9
    adj = dict(lo, adj_c=np.where(on[:, None], lo["adj_c"][row], 0.0), adj_D=np.where(on, lo["adj_D"][row], 0.0))
    # dL/drange divides by the weight of the map's voxel
    e2 = dict(e2, W=np.where(on, ex["W"][row], e2["W"]))
    want_l, want_r, _ = ol.frame_gradients(o2, dict(ranges=near, dirs=dirs, pose=fr["pose"], logits=logits), e2, adj)
    for got, want in ((gl, want_l), (gr, want_r)):
        want = np.asarray(want)
        assert np.all(np.abs(got - want) <= 1e-5 * (np.abs(want) + np.abs(want).max())), np.abs(got - want).max()
    g.close()

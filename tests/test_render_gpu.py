"""Render (slim_render) on the GPU against the oracle's FP64 render of its own
map: where the oracle's sign decisions are clear of ties, hit or miss, the
voxel behind the surface and its label agree exactly and the depth within the
error the D tolerance allows; elsewhere the GPU's answer must be a valid one."""
import numpy as np
import pytest
import torch

import oracle
from oracle.loss import KeyIndex
from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth

from _gpu_util import cuda, integrate_both, make_pair

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sv.load()


@pytest.mark.parametrize("mode", [sv.SEM_CLOSED, sv.SEM_CLOSED_LAST])
def test_render_matches_oracle(mode):
    vs, tau, K = 0.05, 0.15, 5
    print(f"render mode {mode}", flush=True)
    g, o = make_pair(vs, tau, 0.0, 100.0, mode, K)
    for fr in synth.room_sequence(4, seed=5, yaw_span=1.0, width=64, height=48, f=53.3, cx=32.0, cy=24.0):
        integrate_both(g, o, fr["points"], fr["pose"], fr["label"], sv.IN_LABEL_I32)
    pose = synth.pose_matrix(synth.camera_rotation((0.9, 0.35, -0.1)), np.array([2.0312, 1.9687, 1.4219]))
    intr, W, H, near, far = (40.0, 40.0, 39.5, 29.5), 80, 60, 0.05, 6.0
    gout = g.render(pose, intr, W, H, near, far)
    torch.cuda.synchronize()
    oout = oracle.render(o, pose, *intr, W, H, near, far)
    gd, gk, gl = (gout[k].cpu().numpy() for k in ("depth", "key", "label"))
    od, ok, ol, om = oout["depth"], oout["key"], oout["label"], oout["margin"]
    clear = om > 1e-2 * tau
    ghit, ohit = np.isfinite(gd), np.isfinite(od)
    assert np.array_equal(ghit[clear], ohit[clear])
    both = clear & ohit
    assert np.array_equal(gk[both], ok[both])
    assert np.array_equal(gl[both], ol[both])
    assert np.all(gl[~ghit] == -1)
    tol = 2e-6 * od[both] + 1e-5 * tau * np.sqrt(3.0) * vs / om[both] + 1e-6
    err = np.abs(gd[both].astype(np.float64) - od[both])
    print(f"  {both.sum()} clear hits, {(~clear).sum()} near-tie pixels; max depth error {err.max():.2e} m",
          flush=True)
    assert np.all(err <= tol)
    assert both.sum() > 0.5 * W * H
    # near-tie pixels: any GPU surface lies on an observed voxel of the oracle's map
    ex = o.extract()
    idx = KeyIndex(ex["keys"])
    sel = ~clear & ghit
    if sel.any():
        assert np.all(idx.find(gk[sel].reshape(-1, 3)) >= 0)


def test_render_empty_map_and_bad_args():
    g = sv.Map(0.1, 0.3, 0.0, 50.0, sv.SEM_CLOSED, 4, 0, 0, 1 << 10, 1 << 16)
    out = g.render(np.eye(4), (10.0, 10.0, 8.0, 6.0), 16, 12, 0.1, 20.0)
    assert torch.isnan(out["depth"]).all() and (out["label"] == -1).all()
    with pytest.raises(sv.SlimError):
        g.render(np.eye(4), (10.0, 10.0, 8.0, 6.0), 16, 12, 5.0, 1.0)


@pytest.mark.parametrize("W,H,shift", [(1, 1, (0.0, 0.0, 0.0)), (7, 9, (-40.0, 30.0, -7.0)), (33, 17, (0.0, -2.0, -1.5)),
                                       (64, 16, (20000.0, -20000.0, 0.4)), (65, 31, (-3.0, -2.5, 9000.0))])
def test_render_partial_tiles_and_far_maps(W, H, shift):
    """Images that fill their 32 x 16 tiles in part, with an axis-aligned ray among them, over maps on either side of
    the origin and far from it: the oracle's hits, voxels and labels where its decisions are clear."""
    vs, tau, K = 0.05, 0.15, 5
    g, o = make_pair(vs, tau, 0.0, 100.0, sv.SEM_CLOSED, K)
    off = np.asarray(shift)
    for fr in synth.room_sequence(3, seed=6, yaw_span=1.0, width=64, height=48, f=53.3, cx=32.0, cy=24.0):
        pose = fr["pose"].copy()
        pose[:3, 3] += off
        integrate_both(g, o, fr["points"], pose, fr["label"], sv.IN_LABEL_I32)
    pose = synth.pose_matrix(synth.camera_rotation((1.0, 0.0, 0.0)), np.array([2.0312, 1.9687, 1.4219]) + off)
    intr = (0.6 * max(W, 8), 0.6 * max(W, 8), float(W // 2), float(H // 2))
    gout = g.render(pose, intr, W, H, 0.05, 6.0)
    oout = oracle.render(o, pose, *intr, W, H, 0.05, 6.0)
    gd, gk, gl = (gout[k].cpu().numpy() for k in ("depth", "key", "label"))
    od, clear = oout["depth"], oout["margin"] > 1e-2 * tau
    ohit = np.isfinite(od)
    assert np.array_equal(np.isfinite(gd)[clear], ohit[clear])
    both = clear & ohit
    assert np.array_equal(gk[both], oout["key"][both]) and np.array_equal(gl[both], oout["label"][both])
    assert np.all(np.abs(gd[both] - od[both]) <= 2e-6 * od[both] + 1e-5 * tau * np.sqrt(3.0) * vs / oout["margin"][both]
                  + 1e-6)
    assert both.sum() >= (1 if W == 1 else W * H // 4)


def test_render_again_after_growth_and_reset():
    """A map rendered, grown, rendered, reset and filled elsewhere: every image is that of a map which was never
    rendered before, bit for bit, and that of the emptied map holds no surface."""
    frames = synth.room_sequence(4, seed=9, yaw_span=2.0, width=64, height=48, f=53.3, cx=32.0, cy=24.0)

    def fill(m, first, last, shift):
        for fr in frames[first:last]:
            pose = fr["pose"].copy()
            pose[:3, 3] += shift
            m.integrate(torch.from_numpy(fr["points"]).cuda(), pose, torch.from_numpy(fr["label"]).cuda(), sv.IN_LABEL_I32)

    def image(m, shift):
        pose = synth.pose_matrix(synth.camera_rotation((1.0, 0.2, 0.0)), np.array([2.0, 2.0, 1.4]) + shift)
        return m.render(pose, (40.0, 40.0, 32.0, 24.0), 64, 48, 0.05, 8.0)

    def new():
        return sv.Map(0.05, 0.15, 0.0, 100.0, sv.SEM_CLOSED, 5, 0, 0, 1 << 14, 1 << 20)

    def check(got, steps, shift):
        fresh = new()
        for s in steps:
            fill(fresh, *s)
        want = image(fresh, shift)
        for k in want:
            assert torch.equal(got[k].view(torch.int32), want[k].view(torch.int32)), k
        return torch.isfinite(got["depth"]).sum().item()

    g, here, there = new(), np.zeros(3), np.array([55.0, -31.0, 7.0])
    fill(g, 0, 1, here)
    assert check(image(g, here), [(0, 1, here)], here) > 100
    fill(g, 1, 4, here)
    assert check(image(g, here), [(0, 1, here), (1, 4, here)], here) > 100
    g.reset()
    assert not torch.isfinite(image(g, here)["depth"]).any()
    fill(g, 0, 4, there)
    assert check(image(g, there), [(0, 4, there)], there) > 100
    assert not torch.isfinite(image(g, here)["depth"]).any()

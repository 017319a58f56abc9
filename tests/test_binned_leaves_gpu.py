"""Frames whose large leaves are binned before the leaf kernel, against the x-slab items of the batched form (records
bit for bit; the parity tests hold those to the oracle) and the oracle's counts: leaves just below and above the split thresholds, ranges that end inside and between bins, a bin
larger than the leaf kernel's LDS, and every kind of sorted frame."""
import numpy as np
import pytest
import torch

from paper_2512_12945_amd import slimvdb as sv
from _gpu_util import assert_stats_equal, cuda, make_pair

pytestmark = pytest.mark.gpu

VS, TAU = 0.05, 0.15


def points(seed, n, spread):
    """n points on a wall at 1 m: a third evenly over a patch of `spread` metres, a third within one voxel's width of
    its centre, the rest over a wide patch."""
    rng = np.random.default_rng(seed)
    y, z = rng.uniform(-spread, spread, (2, n))
    k = n // 3
    y[:k], z[:k] = rng.uniform(0.011, 0.039, (2, k))
    y[k:2 * k], z[k:2 * k] = rng.uniform(-1.2, 1.2, (2, k))
    p = np.stack([1.0 + rng.normal(0.0, 0.004, n), y, z], axis=1)
    return p[rng.permutation(n)].astype(np.float32)


CASES = [("prob", sv.SEM_CLOSED, 5, 0), ("logit", sv.SEM_CLOSED, 20, 0), ("label", sv.SEM_CLOSED, 40, 0),
         ("label", sv.SEM_CLOSED_LAST, 7, 0), ("bf16", sv.SEM_OPEN, 0, 64), ("f32", sv.SEM_OPEN, 0, 10),
         ("f32", sv.SEM_OPEN_LAST, 0, 10)]


@pytest.mark.parametrize("sem,mode,K,L", CASES)
@pytest.mark.parametrize("n,spread,slab_pairs", [(65537, 0.19, 0), (70001, 0.5, 512)])
def test_binned_equals_slabs(sem, mode, K, L, n, spread, slab_pairs):
    pts = points(n, n, spread)
    rng = np.random.default_rng(n + 1)
    if sem == "label":
        s, kind = rng.integers(0, K, n).astype(np.int32), sv.IN_LABEL_I32
    elif sem in ("prob", "logit"):
        s = rng.standard_normal((n, K)).astype(np.float32)
        kind = sv.IN_LOGIT_F32
        if sem == "prob":
            s, kind = np.abs(s), sv.IN_PROB_F32
    elif sem == "bf16":
        s = (rng.standard_normal((n, L)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
        kind = sv.IN_EMB_BF16
    else:
        s, kind = rng.standard_normal((n, L)).astype(np.float32), sv.IN_EMB_F32
    pose = np.eye(4)
    g, o = make_pair(VS, TAU, 0.0, 10.0, mode, K, L, 1 << 12, 1 << 18)
    b = sv.Map(VS, TAU, 0.0, 10.0, mode, K, L, 0, 1 << 12, 1 << 18)
    for m in (g, b):
        m.set_launch_shape(batch_mode=2, slab_pairs=slab_pairs)
    p, st = cuda(pts), cuda(s)
    for rep in range(2):  # into an empty map, then into the voxels it made
        g.integrate(p, pose, st, kind)
        sv.integrate_batched([b], [dict(points=p, pose=pose, sem=st, kind=kind)])
        assert_stats_equal(g.stats(), o.integrate(pts, pose, s, kind))
        x, y = g.extract(), b.extract()
        for k in x:
            assert torch.equal(x[k].view(torch.int32), y[k].view(torch.int32)), (rep, k)
    g.close()
    b.close()

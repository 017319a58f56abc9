"""The ray walk at the ends of its ranges -- the shortest and the longest band, axis-aligned and diagonal rays, points
nearer than the truncation, cell boundaries met exactly, points on a wave's and a workgroup's edge -- against the oracle:
keys, weights and counts bit for bit."""
import numpy as np
import pytest

from _gpu_util import assert_stats_equal, compare_maps, extract_np, integrate_both, make_pair
from paper_2512_12945_amd import slimvdb as sv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vs,ratio", [(0.1, 1.0), (0.125, 3.0), (0.05, 4.5), (0.125, 6.0), (0.3, 6.0)])
@pytest.mark.parametrize("n", [1, 63, 257, 1500])
@pytest.mark.parametrize("t", [(0.0, 0.0, 0.0), (-77.7, 1234.5, -0.01)])
def test_band(vs, ratio, n, t):
    tau = float(np.float32(vs) * np.float32(ratio))
    rng = np.random.default_rng(n)
    d = rng.standard_normal((n, 3))
    d[::5] = np.eye(3)[rng.integers(0, 3, len(d[::5]))] * rng.choice([-1.0, 1.0], (len(d[::5]), 1))
    d[1::7] = rng.choice([-1.0, 1.0], (len(d[1::7]), 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    r = rng.uniform(0.2 * tau, 40.0 * vs, n)
    r[::3] = np.round(r[::3] / vs) * vs + (r[::3] < vs) * vs
    pose = np.eye(4)
    pose[:3, 3] = t
    g, o = make_pair(vs, tau, 0.0, 100.0, sv.SEM_CLOSED, 3, 0, 1 << 14, 1 << 20)
    for _ in range(2):
        gs, os_ = integrate_both(g, o, (d * r[:, None]).astype(np.float32), pose, rng.integers(-1, 4, n).astype(np.int32),
                                 sv.IN_LABEL_I32)
        assert_stats_equal(gs, os_)
    compare_maps(extract_np(g), o.extract(), tau, sv.SEM_CLOSED, 3, exact_counts=True)
    g.close()

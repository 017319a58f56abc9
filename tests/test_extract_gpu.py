"""Exports around the sizes where the leaf sort changes (a run of 2,048 leaves, 8 runs, 64 runs) and of every kind of
row copy: leaf order, completeness, and the same records as a query gives, bit for bit."""
import numpy as np
import pytest
import torch

from _gpu_util import cuda
from paper_2512_12945_amd import slimvdb as sv

pytestmark = pytest.mark.gpu

VS = 0.125


def leaf_centres(n, seed):
    """n distinct leaf centres around the sensor (the band of one voxel either side stays inside the leaf), shuffled."""
    side = int(np.ceil(n ** (1 / 3))) + 2
    g = np.stack(np.meshgrid(*[np.arange(side) - side // 2] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    g = g[np.abs(g).sum(axis=1) > 1]
    g = g[np.random.default_rng(seed).permutation(len(g))[:n]]
    return ((g + 0.5) * 8 * VS).astype(np.float32)


@pytest.mark.parametrize("n,mode,K,L", [(1, sv.SEM_CLOSED, 20, 0), (2047, sv.SEM_CLOSED, 1, 0), (2048, sv.SEM_OPEN, 0, 3),
                                        (2049, sv.SEM_CLOSED, 5, 0), (16384, sv.SEM_NONE, 0, 0),
                                        (16385, sv.SEM_OPEN_LAST, 0, 33), (131073, sv.SEM_NONE, 0, 0)])
def test_export_order_and_records(n, mode, K, L):
    pts = leaf_centres(n, n)
    rng = np.random.default_rng(n)
    m = sv.Map(VS, VS, 0.0, 1000.0, mode, K, L, 0, 1 << 18, 1 << 25 if mode == sv.SEM_NONE else 1 << 22)
    if K:
        sem, kind = cuda(rng.integers(0, K, n).astype(np.int32)), sv.IN_LABEL_I32
    elif L:
        sem, kind = cuda(rng.standard_normal((n, L)).astype(np.float32)), sv.IN_EMB_F32
    else:
        sem, kind = None, sv.IN_NONE
    m.integrate(cuda(pts), np.eye(4), sem, kind)
    st = m.stats()
    assert st["leaves"] == n
    ex = m.extract()
    assert ex["keys"].shape[0] == st["voxels"]
    k = ex["keys"].long()
    leaf = (k >> 3) + (1 << 17)
    code = ((((leaf[:, 0] << 36) | (leaf[:, 1] << 18) | leaf[:, 2]) << 9) | ((k[:, 0] & 7) << 6) | ((k[:, 1] & 7) << 3)
            | (k[:, 2] & 7))
    assert torch.all(code[1:] > code[:-1])
    assert len(torch.unique(code >> 9)) == n
    q = m.query((ex["keys"].float() + 0.5) * VS)
    no = m.extract(noalloc=True)
    for name in ("D", "W", "sem"):
        assert torch.equal(ex[name], q[name]) and torch.equal(ex[name], no[name]), name
    assert torch.equal(ex["keys"], no["keys"]) and torch.all(ex["W"] > 0)
    m.close()

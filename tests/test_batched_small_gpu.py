"""Batched calls whose maps have fewer ray blocks than the launch has emitting workgroups or items, and more: every map is
bit for bit what calls of its own make it."""
import numpy as np
import pytest
import torch

from _gpu_util import cuda
from paper_2512_12945_amd import slimvdb as sv

pytestmark = pytest.mark.gpu

# points of a map, its mode, classes, embedding size and input
MAPS = [(1, sv.SEM_NONE, 0, 0, sv.IN_NONE), (255, sv.SEM_CLOSED, 20, 0, sv.IN_LABEL_I32),
        (256, sv.SEM_CLOSED, 7, 0, sv.IN_LOGIT_F32), (257, sv.SEM_CLOSED, 30, 0, sv.IN_PROB_F32),
        (0, sv.SEM_CLOSED, 3, 0, sv.IN_LABEL_I32), (2000, sv.SEM_OPEN, 0, 64, sv.IN_EMB_F32),
        (5001, sv.SEM_CLOSED, 20, 0, sv.IN_LOGIT_F32)]


def frame(i, n, K, L, kind, rep):
    rng = np.random.default_rng(100 * i + rep)
    p = rng.uniform(-3.0, 3.0, (n, 3))
    f = dict(points=cuda((p + np.sign(p)).astype(np.float32)), pose=np.eye(4), kind=kind)
    if kind == sv.IN_LABEL_I32:
        f["sem"] = cuda(rng.integers(-1, K, n).astype(np.int32))
    elif kind != sv.IN_NONE:
        f["sem"] = cuda(rng.random((n, K or L), np.float32))
    return f


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("bucket_blocks", [1, 9, 30, 4096])
@pytest.mark.parametrize("use_graph", [False, True])
def test_small_maps(mode, bucket_blocks, use_graph):
    def make():
        return [sv.Map(0.1, 0.3, 0.0, 100.0, m, K, L, 0, 1 << 13, 1 << 20) for _, m, K, L, _ in MAPS]

    batch, alone = make(), make()
    batch[0].set_launch_shape(batch_mode=mode, bucket_blocks=bucket_blocks)
    for rep in range(3):
        frames = [frame(i, n, K, L, kind, rep) for i, (n, _, K, L, kind) in enumerate(MAPS)]
        sv.integrate_batched(batch, frames, use_graph=use_graph)
        for m, f in zip(alone, frames):
            m.integrate(f["points"], f["pose"], f.get("sem"), f["kind"])
    for a, b in zip(batch, alone):
        assert a.stats() == b.stats()
        x, y = a.extract(), b.extract()
        for k in x:
            assert torch.equal(x[k].view(torch.int32), y[k].view(torch.int32)), k
    for m in batch + alone:
        m.close()

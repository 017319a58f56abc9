"""Calls that grow a map's buffers, from one point up, through every form (single, sequence in passes and overlapped,
batched), with exports in between: the map is bit for bit that of single calls into a map whose buffers were large from
the first call."""
import numpy as np
import pytest
import torch

from _gpu_util import cuda
from paper_2512_12945_amd import slimvdb as sv

pytestmark = pytest.mark.gpu


def frame(n, kind, seed):
    rng = np.random.default_rng(seed)
    p = rng.uniform(-5.0, 5.0, (n, 3))
    sem = rng.integers(0, 6, n).astype(np.int32) if kind == sv.IN_LABEL_I32 else rng.random((n, 6), np.float32)
    return dict(points=cuda((p + np.sign(p)).astype(np.float32)), pose=np.eye(4), sem=cuda(sem), kind=kind)


@pytest.mark.parametrize("kind", [sv.IN_LABEL_I32, sv.IN_PROB_F32])
def test_growing_calls(kind):
    a, b = (sv.Map(0.1, 0.3, 0.0, 100.0, sv.SEM_CLOSED, 6, 0, 0, 1 << 15, 1 << 22) for _ in range(2))
    empty = frame(0, kind, 0)
    b.integrate(torch.full((60000, 3), float("nan"), device="cuda"), np.eye(4),
                torch.zeros(60000 * 6, device="cuda").to(empty["sem"].dtype), kind)
    step = 0
    for n in (1, 300, 257, 4000, 700, 20000):
        frames = [frame(max(1, n - 17 * q), kind, 10 * step + q) for q in range(5)]
        if step % 3 == 0:
            for f in frames:
                a.integrate(f["points"], f["pose"], f["sem"], f["kind"])
        elif step % 3 == 1:
            sv.integrate_sequence(a, frames)
        else:
            for f in frames:
                sv.integrate_batched([a], [f])
        for f in frames:
            b.integrate(f["points"], f["pose"], f["sem"], f["kind"])
        x, y = a.extract(), b.extract()
        assert len(x["W"]) > 0
        for k in x:
            assert torch.equal(x[k].view(torch.int32), y[k].view(torch.int32)), (n, k)
        step += 1
    a.close()
    b.close()

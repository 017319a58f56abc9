"""A voxel that the loss lists twice, with its class and with a label outside [0, K): the second adds no cross-entropy term
and takes nothing away, in whichever order.  Loss and gradients are bit for bit those of a list with keys that are not in
the map in its place."""
import numpy as np
import pytest
import torch

from _gpu_util import cuda
from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 3, 15, 16, 32])
def test_listed_twice(K):
    fr = synth.room_frame(seed=K, width=40, height=30, f=30.0, cx=20.0, cy=15.0)
    p = fr["points"].astype(np.float64)
    r = np.linalg.norm(p, axis=1)
    ranges, dirs = cuda(r.astype(np.float32)), cuda((p / r[:, None]).astype(np.float32))
    rng = np.random.default_rng(K)
    logits = cuda(rng.standard_normal((len(r), K)).astype(np.float32))
    g = sv.Map(0.1, 0.3, 0.0, 50.0, sv.SEM_CLOSED, K, 0, 0, 1 << 12, 1 << 18)
    g.integrate_rays(ranges, dirs, fr["pose"], logits, sv.IN_LOGIT_F32)
    keys = g.extract()["keys"]
    M = len(keys)
    samples = ((keys[::3].double() + 0.5) * float(np.float32(0.1))).float()
    y = cuda(rng.integers(0, K, M).astype(np.int32))
    again = cuda(rng.permutation(M)[:M // 2])
    off = cuda(rng.choice([-1, K, K + 7], M // 2).astype(np.int32))
    order = [torch.arange(M + M // 2, device="cuda")]
    order += [order[0].flip(0), cuda(rng.permutation(M + M // 2))]

    def grads(k, lab):
        gl, gr = torch.empty_like(logits), torch.empty_like(ranges)
        g.loss(keys[:5].contiguous(), y[:5].contiguous(), samples)  # leaves other adjoints behind
        loss = g.loss(k.contiguous(), lab.contiguous(), samples).clone()
        g.backward_rays(ranges, dirs, fr["pose"], logits, gl, gr)
        return loss, gl, gr

    for o in order:
        lab = torch.cat([y, off])[o]
        want = grads(torch.cat([keys, keys[again] + 5000])[o], lab)
        assert want[1].abs().max() > 0 or K == 1
        for _ in range(3):
            for a, b in zip(grads(torch.cat([keys, keys[again]])[o], lab), want):
                assert torch.equal(a, b)
    g.close()

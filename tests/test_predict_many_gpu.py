"""The open-set read-out of more points than a launch has lanes for: 2^28 points against a read-out of the few that they
repeat (labels bit for bit)."""
import numpy as np
import pytest
import torch

from _gpu_util import cuda
from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth

pytestmark = pytest.mark.gpu


def test_read_out_of_2_28_points():
    L, P, period = 16, 5, 16 * 1021 + 3
    fr = synth.room_frame(seed=4, width=48, height=36, f=40.0, cx=24.0, cy=18.0)
    rng = np.random.default_rng(2)
    g = sv.Map(0.1, 0.3, 0.0, 100.0, sv.SEM_OPEN, 0, L, 0, 1 << 10, 1 << 17)
    g.integrate(cuda(fr["points"]), fr["pose"], cuda(rng.standard_normal((len(fr["points"]), L)).astype(np.float32)),
                sv.IN_EMB_F32)
    keys = g.extract()["keys"]
    at = ((keys.double() + 0.5) * float(np.float32(0.1))).float()
    at = at[torch.randint(0, len(at), (period,), generator=torch.Generator("cuda").manual_seed(1), device="cuda")]
    at[::7] += 1000.0  # unobserved
    proto = cuda(rng.standard_normal((P, L)).astype(np.float32))
    few = g.predict(at, temperature=0.1, prototypes=proto, prob=False)["label"]
    assert len(few.unique()) == P + 1
    m = 1 << 28
    reps = -(-m // period)
    many = g.predict(at.repeat(reps, 1)[:m].contiguous(), temperature=0.1, prototypes=proto, prob=False)["label"]
    assert torch.equal(many, few.repeat(reps)[:m])
    g.close()

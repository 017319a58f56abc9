"""The open-set read-out of embeddings whose sums lose every later product to rounding when they are formed one after the
other: one component of 2^12, the others 1, so that 2^24 + 1 rounds to 2^24.

Tolerance: two chains of 8 products and their sum, at most L / 64 sums of a wave and the waves' four make a dot product's
and a norm's rounding error at most (10 + L / 64) 2^-24 of |a||b|, the reciprocal norms and the similarity two more;
temperature and softmax double it, and 1e-5 covers the other roundings of a probability.  (One wave a point, with chains
of L / 64 and a tree of 6 levels, lies below that.)"""
import numpy as np
import pytest
import torch

from _gpu_util import cuda
from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth

pytestmark = pytest.mark.gpu

TEMP = 0.02


@pytest.mark.parametrize("L", [512, 1000, 1024])
@pytest.mark.parametrize("P", [2, 9, 20, 130])
def test_long_sums(L, P):
    fr = synth.room_frame(seed=4, width=24, height=17, f=20.0, cx=12.0, cy=8.5)
    n = len(fr["points"])
    a = np.ones(L, np.float32)
    a[0] = 4096.0
    rng = np.random.default_rng(P)
    proto = rng.choice([-1.0, 1.0], (P, L)).astype(np.float32)
    proto[P // 2] = a
    g = sv.Map(0.1, 0.3, 0.0, 100.0, sv.SEM_OPEN, 0, L, 0, 1 << 10, 1 << 15)
    g.integrate(cuda(fr["points"]), fr["pose"], cuda(np.tile(a, (n, 1))), sv.IN_EMB_F32)
    ex = g.extract()
    at = ((ex["keys"].double() + 0.5) * float(np.float32(0.1))).float()
    got = g.predict(at, temperature=TEMP, prototypes=cuda(proto))["prob"].double()
    mean, q = ex["sem"][:, :L].double(), cuda(proto).double()
    want = torch.softmax(mean @ q.T / (mean.norm(dim=1, keepdim=True) * q.norm(dim=1)) / TEMP, dim=1)
    rtol = 2.0 / TEMP * (2 * (10 + L / 64) + 2) * 2.0 ** -24 + 1e-5
    err = float(((got - want).abs() / want).max())
    assert err <= rtol, (err, rtol)
    g.close()

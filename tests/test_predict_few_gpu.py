"""The open-set read-out at the edge between one tile of 16 prototypes and four, with groups of 16 points of which none,
one or all have a record: a point's probabilities, label and variances do not depend on the points it is read with."""
import numpy as np
import pytest
import torch

from _gpu_util import cuda
from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [sv.SEM_OPEN, sv.SEM_OPEN_LAST])
@pytest.mark.parametrize("L", [1, 48, 63, 80, 272, 1024])
@pytest.mark.parametrize("P", [1, 2, 15, 16, 17, 64, 65])
def test_groups(mode, L, P):
    fr = synth.room_frame(seed=5, width=24, height=17, f=20.0, cx=12.0, cy=8.5)
    rng = np.random.default_rng(L + P)
    g = sv.Map(0.1, 0.3, 0.0, 100.0, mode, 0, L, 0, 1 << 10, 1 << 15)
    for _ in range(2):
        e = rng.standard_normal((len(fr["points"]), L)).astype(np.float32)
        g.integrate(cuda(fr["points"]), fr["pose"], cuda(e), sv.IN_EMB_F32)
    ex = g.extract()
    hit = ((ex["keys"].double() + 0.5) * float(np.float32(0.1))).float()[:64]
    miss = hit[:16] + 1000.0
    proto = cuda(rng.standard_normal((P, L)).astype(np.float32))
    opt = dict(temperature=0.1, threshold=0.0, prototypes=proto, var=mode == sv.SEM_OPEN)
    want = g.predict(hit, **opt)
    rec, q = ex["sem"][:64, :L].double(), proto.double()
    sim = rec @ q.T / (rec.norm(dim=1, keepdim=True) * q.norm(dim=1))
    ref = torch.softmax(sim / 0.1, dim=1)
    # chains of at most 10 + L / 64 roundings in a dot product and a norm (twice by the softmax), 1e-5 for the rest
    rtol = 2.0 / 0.1 * (2 * (10 + L / 64) + 2) * 2.0 ** -24 + 1e-5
    assert float(((want["prob"].double() - ref).abs() / ref.clamp_min(1e-30)).max()) <= rtol
    for place in (0, 15):  # one point with a record in each group of 16, then none, then the last group cut short
        at = miss.repeat(67, 1)
        at[place:16 * 64:16] = hit
        at = at[:-9].contiguous()
        got = g.predict(at, **opt)
        here = torch.zeros(len(at), dtype=torch.bool, device="cuda")
        here[place:16 * 64:16] = True
        for k in ("prob", "label") + (("var",) if opt["var"] else ()):
            assert torch.equal(got[k][here].nan_to_num(-1.0) if k != "label" else got[k][here],
                               want[k].nan_to_num(-1.0) if k != "label" else want[k]), k
        assert torch.all(got["prob"][~here] == 0.0) and torch.all(got["label"][~here] == -1)
        if opt["var"]:
            assert torch.isnan(got["var"][~here]).all()
    g.close()

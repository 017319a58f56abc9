"""The open-set read-out at the edges of its tiles (16 or 32 points, 64 prototypes, 16 components, 128 prototypes in LDS)
and with prototypes that are only 4-byte aligned, against a binary64 read-out of the extracted records.

Tolerance: a dot product's or norm's rounding error is at most (chain + 10) 2^-24 of |a||b| for a chain of L / 16
additions, the softmax amplifies a similarity's error by 1 / temperature in two places, and each remaining step of a
probability or a variance is a few roundings (1e-5 covers them)."""
import numpy as np
import pytest
import torch

from _gpu_util import cuda
from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth

pytestmark = pytest.mark.gpu

TEMP = 0.1


@pytest.mark.parametrize("L", [1, 16, 33, 100, 512])
@pytest.mark.parametrize("P,m,aligned", [(1, 1, True), (15, 17, True), (56, 8207, True), (64, 33, False), (65, 47, True),
                                         (128, 8192, True), (129, 15, True), (1024, 31, True)])
def test_read_out_tiles(L, P, m, aligned):
    fr = synth.room_frame(seed=4, width=24, height=17, f=20.0, cx=12.0, cy=8.5)
    n = len(fr["points"])
    rng = np.random.default_rng(L * 1000 + P)
    g = sv.Map(0.1, 0.3, 0.0, 100.0, sv.SEM_OPEN, 0, L, 0, 1 << 10, 1 << 15)
    for _ in range(2):
        g.integrate(cuda(fr["points"]), fr["pose"], cuda(rng.standard_normal((n, L)).astype(np.float32)), sv.IN_EMB_F32)
    ex = g.extract()
    M = ex["keys"].shape[0]
    pick = torch.randint(0, M, (m,), generator=torch.Generator("cuda").manual_seed(P), device="cuda")
    at = ((ex["keys"].double() + 0.5) * float(np.float32(0.1))).float()[pick].clone()
    miss = torch.arange(m, device="cuda") % 5 == 3
    at[miss] += 1000.0
    buf = torch.empty(P * L + 4, device="cuda")
    proto = (buf[:P * L] if aligned else buf[1:1 + P * L]).view(P, L)
    proto.copy_(cuda(rng.standard_normal((P, L)).astype(np.float32)))
    out = g.predict(at, temperature=TEMP, threshold=0.0, prototypes=proto, var=True)
    rec, W = ex["sem"][pick].double(), ex["W"][pick].double()[:, None]
    mean, beta, q = rec[:, :L], rec[:, L:], proto.double()
    sim = (mean @ q.T) / (mean.norm(dim=1, keepdim=True) * q.norm(dim=1))
    want = torch.softmax(sim / TEMP, dim=1)
    want[miss] = 0.0
    rtol = 2.0 / TEMP * (L / 16 + 10) * 2.0 ** -24 + 1e-5
    err = ((out["prob"].double() - want).abs() / want.clamp_min(1e-30)).masked_fill(miss[:, None], 0.0)
    assert torch.all(out["prob"][miss] == 0.0)
    assert float(err.max()) <= rtol, float(err.max())
    var = torch.where((W > 2) & ~miss[:, None], 2.0 * beta * (W + 1.0) / (W * (W - 2.0)), torch.nan)
    assert torch.equal(torch.isnan(var), torch.isnan(out["var"]))
    assert torch.allclose(out["var"].double().nan_to_num(), var.nan_to_num(), rtol=1e-5, atol=0.0)
    top = want.topk(min(2, P), dim=1).values
    clear = ~miss & (top[:, 0] - top[:, -1] > 4 * rtol if P > 1 else True)
    assert torch.all(out["label"][miss] == -1)
    assert torch.equal(out["label"][clear].long(), want.argmax(dim=1)[clear])
    g.close()

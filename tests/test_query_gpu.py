"""slim_query against slim_extract, bit for bit: every length of record that takes another copy of the rows (none,
one float, odd, even, long), point counts around the points a wave takes, misses, repeated points, and an output that
is only 4-byte aligned."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth
from _gpu_util import cuda

pytestmark = pytest.mark.gpu

MODES = [(sv.SEM_NONE, 0, 0), (sv.SEM_CLOSED, 1, 0), (sv.SEM_CLOSED, 5, 0), (sv.SEM_CLOSED, 20, 0), (sv.SEM_CLOSED, 200, 0),
         (sv.SEM_CLOSED_LAST, 4, 0), (sv.SEM_OPEN, 0, 3), (sv.SEM_OPEN, 0, 100), (sv.SEM_OPEN, 0, 1024),
         (sv.SEM_OPEN_LAST, 0, 33)]


@pytest.mark.parametrize("mode,K,L", MODES)
def test_query_equals_extract(mode, K, L):
    fr = synth.room_frame(seed=3, width=24, height=17, f=20.0, cx=12.0, cy=8.5)
    n = len(fr["points"])
    rng = np.random.default_rng(5)
    g = sv.Map(0.1, 0.3, 0.0, 100.0, mode, K, L, 0, 1 << 10, 1 << 15)
    if mode == sv.SEM_NONE:
        sem, kind = None, sv.IN_NONE
    elif K:
        sem, kind = cuda(rng.integers(0, K, n).astype(np.int32)), sv.IN_LABEL_I32
    else:
        sem, kind = cuda(rng.standard_normal((n, L)).astype(np.float32)), sv.IN_EMB_F32
    g.integrate(cuda(fr["points"]), fr["pose"], sem, kind)
    ex = g.extract()
    M, S = ex["keys"].shape[0], g.nsem
    centres = ((ex["keys"].double() + 0.5) * float(np.float32(0.1))).float()
    for m in (1, 3, 5, 15, 17, 65, M):
        pick = torch.randint(0, M, (m,), generator=torch.Generator("cuda").manual_seed(m), device="cuda")
        at = centres[pick].clone()
        miss = torch.arange(m, device="cuda") % 7 == 4
        at[miss] += 1000.0
        want = {k: torch.where(miss.view(-1, *[1] * (ex[k].dim() - 1)), 0.0, ex[k][pick]) for k in ("D", "W", "sem")}
        got = g.query(at)
        for k in want:
            assert torch.equal(got[k], want[k]), (m, k)
        if S:
            # rows at a 4-byte aligned address, and nothing written before or after them
            d, w = torch.empty(m, device="cuda"), torch.empty(m, device="cuda")
            buf = torch.full((m * S + 2,), -7.0, device="cuda")
            sv._check(g._L.slim_query(g.h, sv._ptr(at), m, sv._ptr(d), sv._ptr(w),
                                      ctypes.c_void_p(buf.data_ptr() + 4), sv._stream(g.device)))
            assert torch.equal(buf[1:-1].view(m, S), want["sem"])
            assert buf[0] == -7.0 and buf[-1] == -7.0
    g.close()

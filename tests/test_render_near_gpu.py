"""Renders of rays too short for the filters of empty space, on either side of that line, before and after the map grows
and is emptied: a surface that both ranges reach is the same bit for bit, and images equal those of a map that was not
rendered before."""
import numpy as np
import pytest
import torch

from paper_2512_12945_amd import slimvdb as sv
from paper_2512_12945_amd import synth

pytestmark = pytest.mark.gpu

VS, NEAR = 0.05, 0.25
INTR = (40.0, 40.0, 31.5, 23.5)


def new_map():
    return sv.Map(VS, 0.15, 0.0, 100.0, sv.SEM_CLOSED, 5, 0, 0, 1 << 13, 1 << 18)


def fill(m, frames, shift=0.0):
    for fr in frames:
        pose = fr["pose"].copy()
        pose[:3, 3] += shift
        m.integrate(torch.from_numpy(fr["points"]).cuda(), pose, torch.from_numpy(fr["label"]).cuda(), sv.IN_LABEL_I32)


def image(m, cells, shift=0.0):
    pose = synth.pose_matrix(synth.camera_rotation((1.0, 0.2, -0.3)), np.array([2.0, 2.0, 1.4]) + shift)
    out = m.render(pose, INTR, 64, 48, NEAR, NEAR + cells * VS)
    return {k: v.clone() for k, v in out.items()}


def same(a, b, on=None):
    on = torch.ones_like(a["label"], dtype=torch.bool) if on is None else on
    return all(torch.equal(a[k][on].view(torch.int32), b[k][on].view(torch.int32)) for k in a)


def test_short_rays():
    frames = synth.room_sequence(4, seed=9, yaw_span=2.0, width=64, height=48, f=53.3, cx=32.0, cy=24.0)
    m = new_map()
    fill(m, frames[:2])
    hits = []
    for cells in (1, 20, 47.5, 48.5, 64, 160):  # 48 cells is the line
        out, long = image(m, cells), image(m, 200)
        reach = NEAR + (cells - 2) * VS
        on = torch.isfinite(long["depth"]) & (long["depth"] < reach)
        assert same(out, long, on)
        # what only the longer rays see lies at the end of the shorter ones or behind
        only = torch.isfinite(long["depth"]) & ~torch.isfinite(out["depth"])
        assert torch.all(long["depth"][only] >= reach)
        assert torch.all(torch.isfinite(long["depth"][torch.isfinite(out["depth"])]))
        hits.append(int(on.sum()))
    assert hits[0] == 0 and 0 < hits[2] <= hits[3] < hits[-1]
    # growth after short and long renders, then a new start elsewhere
    fill(m, frames[2:])
    for cells in (40, 160):
        f = new_map()
        fill(f, frames)
        assert same(image(m, cells), image(f, cells))
    m.reset()
    assert torch.isnan(image(m, 40)["depth"]).all() and torch.isnan(image(m, 160)["depth"]).all()
    fill(m, frames[:3], 12.0)
    f = new_map()
    fill(f, frames[:3], 12.0)
    for cells in (160, 40, 160):
        assert same(image(m, cells, 12.0), image(f, cells, 12.0))


def test_growth_inside_a_graph():
    """A captured render replayed after the map has grown twice shows the grown map."""
    frames = synth.room_sequence(4, seed=9, yaw_span=2.0, width=64, height=48, f=53.3, cx=32.0, cy=24.0)
    m = new_map()
    pose = synth.pose_matrix(synth.camera_rotation((1.0, 0.2, -0.3)), np.array([2.0, 2.0, 1.4]))
    out = {}
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        m.render(pose, INTR, 64, 48, NEAR, 8.0)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            out = m.render(pose, INTR, 64, 48, NEAR, 8.0)
        for k in range(4):
            fill(m, frames[k:k + 1])
            graph.replay()
            f = new_map()
            fill(f, frames[:k + 1])
            assert same(out, f.render(pose, INTR, 64, 48, NEAR, 8.0))
    torch.cuda.synchronize()

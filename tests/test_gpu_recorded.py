"""Steps that the caller records into a HIP graph of its own.  dmr_step only
queues launches between growth tests, so any stretch of steps that holds none
can be recorded, the first after a creation, a growth or a load included."""
import numpy as np
import pytest

from paper_2105_13276_amd import binding as B
from paper_2105_13276_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("hz", "ex", "ey", "jx", "jy", "n", "acc", "ring")


def _record(sim, n):
    """n steps of sim as a graph (nothing has run yet)."""
    import torch
    g = torch.cuda.CUDAGraph()
    g.capture_begin(capture_error_mode="thread_local")
    try:
        sim.step(n)
    finally:
        g.capture_end()
    return g


def _same(a, b):
    for lv in (0, 1) if a.cfg["mode"] != "uniform" else (0,):
        for f in FIELDS:
            x, y = a.get(f, lv), b.get(f, lv)
            assert np.array_equal(x, y), (lv, f, int((x != y).sum()))


def _union():
    cfg = W.make(256, 160, 32, "dynamic", 1, erms_over_ebd=3.0, regrid_rule="union")
    dx = W.C0 / 110e9 / 32
    return cfg, W.seeds(cfg, [(0.4 * 256 * dx, 0.3 * 160 * dx)], [1e17])


@pytest.mark.parametrize("split_min", [None, "0"])
def test_first_steps_of_a_union_level(split_min, monkeypatch):
    """The first recorded step after the level came about: created, grown by
    blocks, loaded; on a grid whose steps are split around the level and on
    one whose are not."""
    import torch
    cfg, (sb, sf) = _union()
    if split_min:
        monkeypatch.setenv("DMR_SPLIT_MIN", split_min)
    with torch.cuda.stream(torch.cuda.Stream()):
        s, ref = B.Sim(cfg, sb, sf), B.Sim(cfg, sb, sf)
        for change in ("created", "grown", "loaded"):
            if change == "grown":
                mask = np.zeros_like(s.blocks())
                mask[6, 11] = 1
                s.add_blocks(mask)
                ref.add_blocks(mask)
            if change == "loaded":
                s.load(s.save())
            g = _record(s, 11)
            g.replay()
            ref.step(11)
            _same(s, ref)
        s.sync()
        ref.sync()

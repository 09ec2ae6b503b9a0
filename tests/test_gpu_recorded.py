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


def _replayable(kind):
    """No source (whose values a graph would hold as they were when recorded)
    but given fields: a period's graph can run again and again."""
    if kind in ("uniform", "uniform_no_continuity"):
        cfg = W.make(200, 90, 32, "uniform", 1, tfsf_i=0, continuity_on=kind == "uniform")
    elif kind == "r4":
        cfg = W.make(160, 112, 32, "static", 1, r=4, block=8, tfsf_i=0, static_ext=(70, 40, 90, 61))
    else:
        cfg = W.make(256, 160, 32, "static", 1, tfsf_i=0, static_ext=(112, 64, 144, 96),
                     regrid_rule="union" if kind == "union" else "blocks")
    nx, ny = cfg["nx"], cfg["ny"]
    g = np.random.Generator(np.random.PCG64(nx + ny))
    base = 10.0 ** g.uniform(17, 20, (ny + 1, nx + 1))
    fields = {f: 4e6 * g.uniform(-1, 1, d) for f, d in
              (("ex", (ny + 1, nx)), ("ey", (ny, nx + 1)))}
    return cfg, base, fields


@pytest.mark.parametrize("kind,n,start", [
    ("uniform", 64, 3), ("uniform_no_continuity", 8, 0), ("rect", 64, 3), ("rect", 64, 0),
    ("r4", 64, 5), ("union", 64, 3)])
def test_a_recorded_stretch_runs_again(kind, n, start, monkeypatch):
    """A graph of a whole period (without continuity: of an even number of
    steps), replayed in a row and between steps of the handle itself, is those
    steps each time, wherever in a window block it starts."""
    import torch
    cfg, base, fields = _replayable(kind)
    monkeypatch.setenv("DMR_SPLIT_MIN", "0")
    warm = 6 * cfg["steps_per_period"] + start
    with torch.cuda.stream(torch.cuda.Stream()):
        s, ref = B.Sim(cfg, base, None), B.Sim(cfg, base, None)
        for q in (s, ref):
            for f, v in fields.items():
                q.set(f, 0, v)
            q.step(warm)
        g = _record(s, n)
        for again, eager in ((1, n), (3, n), (1, 5), (0, n - 5), (2, 0)):
            for _ in range(again):
                g.replay()
            s.step(eager)
            ref.step(again * n + eager)
            if eager != 5:
                _same(s, ref)
            torch.zeros(1000, device="cuda").sum().item()  # other work between
        s.sync()
        ref.sync()


def test_a_recorded_stretch_of_a_batch_runs_again():
    """The same of a tuned batch; then whole intervals from the batch's graph."""
    import torch
    cfgs, sims = [], []
    with torch.cuda.stream(torch.cuda.Stream()):
        for nx, ny in ((512, 256), (640, 448)):
            cfgs.append(W.make(nx, ny, 32, "static", 1, tfsf_i=0,
                               static_ext=(nx // 2 - 16, ny // 2 - 8, nx // 2 + 16, ny // 2 + 8)))
        seeds = [W.seeds(c) for c in cfgs]
        b = B.Batch(cfgs, seeds)
        sims = [B.Sim(c, *q) for c, q in zip(cfgs, seeds)]
        for k, c in enumerate(cfgs):
            e = np.random.Generator(np.random.PCG64(k)).uniform(-4e6, 4e6, (c["ny"], c["nx"] + 1))
            B.Sim.set(b.instances[k], "ey", 0, e)
            sims[k].set("ey", 0, e)
        b.step(512 + 3)
        for s in sims:
            s.step(512 + 3)
        g = torch.cuda.CUDAGraph()
        g.capture_begin(capture_error_mode="thread_local")
        try:
            b.step(64)
        finally:
            g.capture_end()
        for again, eager in ((2, 64), (1, 0), (1, 61), (0, 576)):
            for _ in range(again):
                g.replay()
            b.step(eager)
            b.sync()
            for h, s in zip(b.instances, sims):
                s.step(64 * again + eager)
                _same(h, s)
        b.close()

"""Several base-level steps in one launch (no patch, or away from it) against
one launch per step: the same operations on every entity, so the same bits.
Sizes around the block shape (64 columns, 4 rows a wave): grids smaller than
a halo, one row or column more than whole blocks, the last block owning only
the outer row or column; walls of both kinds; the source column at either
end and none."""
import os

import numpy as np
import pytest

from paper_2105_13276_amd import binding as B
from paper_2105_13276_amd import workloads as W

FIELDS = ("hz", "ex", "ey", "jx", "jy", "n", "acc", "ring")


def _run(cfg, base, fields, multi, chunks):
    old = os.environ.get("DMR_MULTI")
    os.environ["DMR_MULTI"] = multi
    try:
        s = B.Sim(cfg, base, None)
    finally:
        if old is None:
            os.environ.pop("DMR_MULTI")
        else:
            os.environ["DMR_MULTI"] = old
    for f, v in fields.items():
        s.set(f, 0, v)
    got = []
    for n in chunks:
        s.step(n)
        got.append({f: s.get(f, 0) for f in FIELDS})
    # Hz of the half level before is part of a saved state
    state = s.save(np.zeros(s.state_bytes(), np.uint8))
    s.sync()
    s.close()
    return got, state


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny,cpl,bc_x,bc_y,src,multi", [
    (4, 4, 4, "mur", "mur", 1, "8"),
    (5, 17, 16, "pec", "mur", 4, "8,5"),
    (48, 96, 32, "mur", "pec", 8, "8,12"),      # last blocks: column 48, row 96 alone
    (47, 95, 32, "mur", "mur", 46, "8,8"),      # whole blocks
    (97, 33, 36, "mur", "mur", 9, "8"),         # window block of 9 steps: 5 + 4
    (64, 64, 64, "pec", "pec", 0, "8,16"),
    (200, 61, 44, "mur", "pec", 199, "3,6"),
    (333, 260, 16, "pec", "mur", 4, "8,8"),
])
def test_several_steps_in_one_launch(nx, ny, cpl, bc_x, bc_y, src, multi):
    cfg = W.make(nx, ny, cpl, "uniform", 1, bc_x=bc_x, bc_y=bc_y, tfsf_i=src)
    g = np.random.Generator(np.random.PCG64(nx * 1000 + ny))
    base = 10.0 ** g.uniform(17, 20, (ny + 1, nx + 1))
    E = 4e6
    fields = dict(hz=E / 377 * g.uniform(-1, 1, (ny, nx)), ex=E * g.uniform(-1, 1, (ny + 1, nx)),
                  ey=E * g.uniform(-1, 1, (ny, nx + 1)))
    chunks = (1, 23, cpl + 5)  # an odd place in a window block, then past a period
    a, sa = _run(cfg, base, fields, multi, chunks)
    b, sb = _run(cfg, base, fields, "1", chunks)
    for x, y in zip(a, b):
        for f in FIELDS:
            assert np.array_equal(x[f], y[f]), (f, int((x[f] != y[f]).sum()))
    # the header's unused bytes apart; as numbers (a PEC zero may be -0)
    assert np.array_equal(sa[:72], sb[:72])
    assert np.array_equal(sa[256:].view(np.float32), sb[256:].view(np.float32))


def _refined(kind):
    lam = W.C0 / 110e9
    if kind == "r4":
        cfg = W.make(160, 112, 16, "dynamic", 1, r=4, block=8, erms_over_ebd=3.0)
    else:
        cfg = W.make(256, 160, 32, "dynamic", 1, erms_over_ebd=3.0,
                     regrid_rule="union" if kind == "union" else "blocks")
    if kind == "static":  # a patch off the block lines, two cells from the wall margin
        cfg.update(mode="static", static_ext=(101, 17, 140, 41))
    if kind == "wide":    # too large a share of the grid: one launch a step
        cfg.update(mode="static", static_ext=(30, 20, 240, 140))
    cfg["regrid_every"] = 4 * (cfg["steps_per_period"] // 8)
    dx = lam / cfg["cells_per_lambda"]
    at = [(0.55, 0.4)] if kind != "union" else [(0.4, 0.3), (0.75, 0.7)]
    centres = [(x * cfg["nx"] * dx, y * cfg["ny"] * dx) for x, y in at]
    return cfg, W.seeds(cfg, centres, [1e17] * len(at))


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["rect", "r4", "union", "static", "wide"])
def test_steps_split_around_the_fine_level(kind, monkeypatch):
    """Groups of steps split into the cells around the fine level (one launch a
    step) and the rest (one launch a group) against one launch per step, over
    growths, with stretches that end inside a window block: the same bits on
    both levels, also after a restart."""
    cfg, (sb, sf) = _refined(kind)
    runs = []
    for env in ({"DMR_MULTI": "1"}, {"DMR_SPLIT_MIN": "0"}, {"DMR_SPLIT_MIN": "0", "DMR_MULTI": "3"}):
        for k in ("DMR_MULTI", "DMR_SPLIT_MIN"):
            monkeypatch.delenv(k, raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        s = B.Sim(cfg, sb, sf)
        got = []
        for n in (5, 100, 61):
            s.step(n)
            got.append({(f, lv): s.get(f, lv) for lv in (0, 1) for f in FIELDS})
            got[-1]["patch"] = np.array(s.patch())
        s.load(s.save())
        s.step(30)
        got.append({(f, lv): s.get(f, lv) for lv in (0, 1) for f in FIELDS})
        s.sync()
        runs.append(got)
    for other in runs[1:]:
        for x, y in zip(runs[0], other):
            for f in x:
                assert np.array_equal(x[f], y[f]), f


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["rect", "r4", "union", "static", "wide"])
def test_periods_from_a_graph(kind, monkeypatch):
    """Whole periods of a refined run replayed from one graph against launch by
    launch: over growth tests at a period's end and inside one, stretches that
    start and end inside a period, eager work and reads between the replays,
    and a restart: the same bits and saved states."""
    cfg, (sb, sf) = _refined(kind)
    K = cfg["steps_per_period"]
    for every in (4 * (K // 8), 2 * K):
        cfg["regrid_every"] = every
        runs = []
        for env in ("0", "1"):
            monkeypatch.setenv("DMR_PERIOD", env)
            s = B.Sim(cfg, sb, sf)
            got = []
            for n in (K + 3, 6 * K, 3, 2 * K - 6, 5 * K, K, K):
                s.step(n)
                got.append({(f, lv): s.get(f, lv) for lv in (0, 1) for f in FIELDS})
                got[-1]["patch"] = np.array(s.patch())
            got[-1]["state"] = s.save(np.zeros(s.state_bytes(), np.uint8))[256:]
            s.load(s.save())
            s.step(4 * K + 5)
            got.append({(f, lv): s.get(f, lv) for lv in (0, 1) for f in FIELDS})
            s.sync()
            s.close()
            runs.append(got)
        for x, y in zip(*runs):
            assert x.keys() == y.keys()
            for f in x:
                assert np.array_equal(x[f], y[f]), f


@pytest.mark.gpu
def test_periods_while_the_caller_records():
    """A period whose stream the caller is recording goes launch by launch into
    the caller's graph: replayed, it gives the bits of the steps themselves."""
    import torch
    cfg, (sb, sf) = _refined("static")
    K = cfg["steps_per_period"]
    with torch.cuda.stream(torch.cuda.Stream()):
        s, ref = B.Sim(cfg, sb, sf), B.Sim(cfg, sb, sf)
        for q in (s, ref):
            q.step(6 * K)
            q.sync()
        g = torch.cuda.CUDAGraph()
        g.capture_begin(capture_error_mode="thread_local")
        s.step(K)
        g.capture_end()
        g.replay()
        ref.step(K)
        for f in FIELDS:
            for lv in (0, 1):
                assert np.array_equal(s.get(f, lv), ref.get(f, lv)), f
        s.sync()


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["rect", "r4", "union"])
def test_batch_steps_split_around_the_fine_levels(kind, monkeypatch):
    """A batch whose steps are split (tuned configuration, a captured interval,
    stretches that leave an odd number of groups) against plain runs of one
    launch per step: the same bits and saved states."""
    lam = W.C0 / 110e9
    cfgs, seeds = [], []
    for nx, ny in ((384, 224), (320, 256), (256, 288)):
        if kind == "r4":
            cfg = W.make(nx, ny, 32, "dynamic", 1, r=4, block=16, erms_over_ebd=2.0)
        else:
            cfg = W.make(nx, ny, 32, "dynamic", 1, erms_over_ebd=2.0,
                         regrid_rule="union" if kind == "union" else "blocks")
        dx = lam / 32
        cfgs.append(cfg)
        seeds.append(W.seeds(cfg, [(0.5 * nx * dx, 0.45 * ny * dx)], [1e17]))
    b = B.Batch(cfgs, seeds)
    monkeypatch.setenv("DMR_MULTI", "1")
    plain = [B.Sim(c, *s) for c, s in zip(cfgs, seeds)]
    monkeypatch.delenv("DMR_MULTI")
    for n in (256, 264, 504, 3):
        b.step(n)
        for h, s in zip(b.instances, plain):
            s.step(n)
            assert h.patch() == s.patch()
            for lv in (0, 1):
                for f in FIELDS:
                    assert np.array_equal(h.get(f, lv), s.get(f, lv)), (n, f, lv)
            a, c = (x.save(np.zeros(x.state_bytes(), np.uint8)) for x in (h, s))
            assert np.array_equal(a[256:].view(np.float32), c[256:].view(np.float32))
    b.sync()
    b.close()


@pytest.mark.gpu
@pytest.mark.parametrize("w,h,x,y,waves,gamma", [
    (1, 1, 40, 30, 8, 1e-3),       # smaller than a halo
    (3, 25, 41, 31, 16, 1e-3),     # 50 own columns or rows: one more node than whole blocks
    (25, 2, 33, 20, 12, 1e-3),
    (24, 8, 60, 41, 12, 0.0),      # whole blocks less one node; no filter
    (60, 57, 30, 20, 0, 1.0 / 64),
    (101, 33, 30, 20, 8, 1e-3),
])
def test_register_patch_tiles(w, h, x, y, waves, gamma, monkeypatch):
    """Both r = 2 substeps in the register tiles against one launch a substep,
    over patches of sizes around the tiles' own 50 columns and 18 to 50 rows:
    the same bits on both levels."""
    cfg = W.make(160, 96, 32, "static", 1, static_ext=(x, y, x + w, y + h), fine_filter=gamma,
                 erms_over_ebd=3.0)
    g = np.random.Generator(np.random.PCG64(w * 100 + h))
    base = 10.0 ** g.uniform(17, 20, (97, 161))
    E = 4e6
    runs = []
    for env in ({"DMR_FINE_REG": "0,%d" % waves}, {"DMR_FUSE": "0", "DMR_MULTI": "1"}):
        for k in ("DMR_FINE_REG", "DMR_FUSE", "DMR_MULTI"):
            monkeypatch.delenv(k, raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        s = B.Sim(cfg, base, None)
        q = np.random.Generator(np.random.PCG64(7))
        for lv in (0, 1):
            for f in ("hz", "ex", "ey"):
                a = E * q.uniform(-1, 1, s.dims(f, lv))
                s.set(f, lv, a / 377 if f == "hz" else a)
        got = []
        for n in (1, 3, 70):
            s.step(n)
            got.append({(f, lv): s.get(f, lv) for lv in (0, 1) for f in FIELDS})
        s.sync()
        runs.append(got)
    for a, b in zip(*runs):
        for f in a:
            assert np.array_equal(a[f], b[f]), (f, int((a[f] != b[f]).sum()))


@pytest.mark.gpu
@pytest.mark.parametrize("ny", [4, 5, 6, 7, 255])
def test_fields_read_back_as_written(ny):
    """Read-out in groups of rows: every remainder of the row count."""
    cfg = W.make(257, ny, 16, "uniform", 1)
    s = B.Sim(cfg, None, None)
    g = np.random.Generator(np.random.PCG64(ny))
    for f in ("ex", "ey"):
        v = g.uniform(-1, 1, s.dims(f, 0)).astype(np.float32)
        s.set(f, 0, v)
        assert np.array_equal(s.get(f, 0), v) and np.array_equal(s.get_device(f, 0).cpu(), v)
    s.close()


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(592, 448), (1040, 256), (528, 512)])
def test_continuity_rows_of_a_plain_run_and_a_batch(nx, ny):
    """The base level's continuity with two rows a thread (plain run of 2^18
    nodes and more; 449, 257 and 513 rows of nodes) against the batch's four
    rows a thread, and both levels' window: the same bits."""
    cfg = W.make(nx, ny, 16, "dynamic", 1, erms_over_ebd=2.0)
    dx = W.C0 / 110e9 / 16
    seeds = W.seeds(cfg, [(0.6 * nx * dx, 0.5 * ny * dx)], [1e17])
    s, b = B.Sim(cfg, *seeds), B.Batch([cfg], [seeds])
    for n in (33, 64):
        s.step(n)
        b.step(n)
        b.sync()
        for f, lv in (("n", 0), ("erms2", 0), ("ring", 0), ("n", 1)):
            assert np.array_equal(s.get(f, lv), b.instances[0].get(f, lv)), f
    s.close()
    b.close()


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny,bc_x,bc_y", [(97, 70, "pec", "pec"), (97, 70, "mur", "mur"),
                                             (64, 48, "pec", "mur"), (47, 33, "mur", "pec")])
@pytest.mark.parametrize("multi", ["8", "5,6"])
def test_walls_of_several_steps_bit_by_bit(nx, ny, bc_x, bc_y, multi, monkeypatch):
    """Every bit of every field and of the saved state, the sign of zeros on
    the walls among them, and with infinite values beside the walls, against
    one launch a step: walls stay +0, nothing outside the grid reaches it."""
    cfg = W.make(nx, ny, 16, "uniform", 1, bc_x=bc_x, bc_y=bc_y, tfsf_i=4)
    g = np.random.Generator(np.random.PCG64(nx + ny))
    base = 10.0 ** g.uniform(17, 20, (ny + 1, nx + 1))
    E = 4e6
    fields = dict(hz=E / 377 * g.uniform(-1, 1, (ny, nx)), ex=E * g.uniform(-1, 1, (ny + 1, nx)),
                  ey=E * g.uniform(-1, 1, (ny, nx + 1)))
    for infinite in (False, True):
        if infinite:
            for j, i in ((0, 20), (ny - 1, 30), (20, 0), (25, nx - 1), (0, 0), (ny - 1, nx - 1)):
                fields["hz"][j, i] = np.inf
        runs = []
        for env in (multi, "1"):
            monkeypatch.setenv("DMR_MULTI", env)
            s = B.Sim(cfg, base, None)
            for f, v in fields.items():
                s.set(f, 0, v)
            got = []
            for n in (3, 8, 30):
                s.step(n)
                got.append({f: s.get(f, 0) for f in FIELDS})
            runs.append((got, s.save(np.zeros(s.state_bytes(), np.uint8))))
            s.close()
        (a, sa), (b, sb) = runs
        for x, y in zip(a, b):
            for f in FIELDS:
                nan = np.isnan(x[f])
                assert np.array_equal(nan, np.isnan(y[f])), (f, infinite)
                assert np.array_equal(x[f].view(np.uint32)[~nan], y[f].view(np.uint32)[~nan]), f
        if not infinite:
            assert np.array_equal(sa, sb)
        nan = np.isnan(sa[256:].view(np.float32))
        assert np.array_equal(nan, np.isnan(sb[256:].view(np.float32)))
        assert np.array_equal(sa[256:].view(np.uint32)[~nan], sb[256:].view(np.uint32)[~nan])


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["rect", "r4", "union", "wall"])
@pytest.mark.parametrize("bc_x,bc_y", [("pec", "pec"), ("mur", "pec")])
def test_split_steps_between_walls_with_the_full_source(kind, bc_x, bc_y, monkeypatch):
    """Split steps with conducting walls, also within the reach of the fine level
    (wall), and the Townsend source with recombination: the bits of one launch
    a step, saved states included."""
    cfg, (sb, sf) = _refined("static" if kind == "wall" else kind)
    cfg.update(bc_x=bc_x, bc_y=bc_y, source_model="townsend", beta_rec=2e-13)
    if kind == "wall":
        cfg["static_ext"] = (200, 3, 253, 40)
    runs = []
    for env in ("1", "8", "5"):
        monkeypatch.setenv("DMR_MULTI", env)
        monkeypatch.setenv("DMR_SPLIT_MIN", "0")
        s = B.Sim(cfg, sb, sf)
        got = []
        for n in (5, 130, 61):
            s.step(n)
            got.append({(f, lv): s.get(f, lv) for lv in (0, 1) for f in FIELDS})
        runs.append((got, s.save(np.zeros(s.state_bytes(), np.uint8))))
        s.sync()
        s.close()
    for got, state in runs[1:]:
        for x, y in zip(runs[0][0], got):
            for f in x:
                assert np.array_equal(x[f].view(np.uint32), y[f].view(np.uint32)), f
        assert np.array_equal(state, runs[0][1])

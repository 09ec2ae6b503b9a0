"""Limits of the workspace: what does not fit is refused, and what fitted
before the several-step forms had planes of their own still does."""
import numpy as np
import pytest

from paper_2105_13276_amd import binding as B
from paper_2105_13276_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,fits", [(4, 4, False), (20, 20, False), (63, 31, False),
                                        (63, 32, True), (64, 20, True)])
def test_weighted_sum_needs_its_staging_area(nx, ny, fits):
    """The 1025 partial sums go to the staging plane (64 floats a row up to 63
    cells, 128 up to 127): a grid whose plane is smaller is refused, and
    nothing beyond the plane (the live Hz of an earlier half level among it)
    is written."""
    cfg = W.make(nx, ny, 4, "uniform", 1)
    s = B.Sim(cfg, np.full((ny + 1, nx + 1), 1e18), None)
    s.step(11)
    before = s.save(np.zeros(s.state_bytes(), np.uint8))
    w = np.ones((ny + 1, nx + 1), np.float32)
    if fits:
        n = s.get("n", 0).astype(np.float64)
        assert abs(s.weighted_sum(w) - n.sum()) <= 1e-12 * n.sum()
    else:
        with pytest.raises(B.DmrError, match="ENOMEM"):
            s.weighted_sum(w)
    assert np.array_equal(s.save(np.zeros(s.state_bytes(), np.uint8)), before)
    s.close()


FIELDS = ("hz", "ex", "ey", "jx", "jy", "n", "acc", "ring")

# configuration, and the bytes of two levels' 21 planes, the staging plane, the
# block arrays and (union) the tile lists alone
SMALLEST = [
    (dict(nx=256, ny=128, cells_per_lambda=64), 3633920),
    (dict(nx=512, ny=256, cells_per_lambda=32, mode="dynamic"), 61556480),
    (dict(nx=160, ny=112, cells_per_lambda=16, mode="dynamic", r=4, block=8), 30906880),
    (dict(nx=256, ny=160, cells_per_lambda=32, mode="dynamic", regrid_rule="union"), 21190656),
    (dict(nx=640, ny=448, cells_per_lambda=32, mode="dynamic"), 132653056),
]


def _seeds(cfg):
    dx = W.C0 / 110e9 / cfg["cells_per_lambda"]
    return W.seeds(cfg, [(0.6 * cfg["nx"] * dx, 0.5 * cfg["ny"] * dx)], [1e17])


@pytest.mark.parametrize("kw,nbytes", SMALLEST)
def test_smallest_workspace(kw, nbytes, monkeypatch):
    """Without the planes and tables of several steps a launch, split steps and
    recorded periods: one launch a step, the same bits.  One byte less is
    refused."""
    cfg = W.make(periods=1, erms_over_ebd=2.0, **kw)
    seeds = _seeds(cfg)
    ref = B.Sim(cfg, *seeds)
    assert B.workspace_bytes(cfg) > nbytes
    monkeypatch.setattr(B, "workspace_bytes", lambda c: nbytes - 1)
    with pytest.raises(B.DmrError, match="ENOMEM"):
        B.Sim(cfg, *seeds)
    monkeypatch.setattr(B, "workspace_bytes", lambda c: nbytes)
    s = B.Sim(cfg, *seeds)
    for n in (5, 200, 61):
        s.step(n)
        ref.step(n)
        for lv in (0, 1) if cfg["mode"] != "uniform" else (0,):
            for f in FIELDS:
                assert np.array_equal(s.get(f, lv), ref.get(f, lv)), (n, f, lv)
    s.sync()
    s.close()
    ref.close()


def test_smallest_workspace_of_a_batch(monkeypatch):
    cfgs = [W.make(nx, nx // 2, 32, "dynamic", 1, erms_over_ebd=2.0) for nx in (128, 192)]
    seeds = [_seeds(c) for c in cfgs]
    plain = [B.Sim(c, *s) for c, s in zip(cfgs, seeds)]
    lib, size = B.lib(), [14428672]

    class Lib:  # the library, but for the size it asks for
        def __getattr__(self, name):
            return getattr(lib, name)

        def dmr_batch_workspace_bytes(self, p, n, out):
            lib.dmr_batch_workspace_bytes(p, n, out)
            assert out._obj.value > size[0]
            out._obj.value = size[0]
            return 0

    monkeypatch.setattr(B, "lib", Lib)
    b = B.Batch(cfgs, seeds)
    for n in (256, 264, 504, 3):
        b.step(n)
        b.sync()
        for h, s in zip(b.instances, plain):
            s.step(n)
            for lv in (0, 1):
                for f in FIELDS:
                    assert np.array_equal(h.get(f, lv), s.get(f, lv)), (n, f, lv)
    b.close()
    size[0] -= 4096
    with pytest.raises(B.DmrError, match="ENOMEM"):
        B.Batch(cfgs, seeds)

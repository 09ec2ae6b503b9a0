"""Whether a batch splits its steps around the fine levels: as timed, or by
size; the same bits either way."""
import numpy as np
import pytest

from paper_2105_13276_amd import binding as B
from paper_2105_13276_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("hz", "ex", "ey", "jx", "jy", "n", "acc", "ring")


def _batch(sizes, kind="rect", field=2.0):
    cfgs, seeds = [], []
    for nx, ny in sizes:
        kw = {"rect": {}, "r4": dict(r=4), "union": dict(regrid_rule="union"),
              "union8": dict(regrid_rule="union", block=8)}[kind]
        cfg = W.make(nx, ny, 32, "dynamic", 1, erms_over_ebd=field, **kw)
        dx = W.C0 / 110e9 / 32
        cfgs.append(cfg)
        seeds.append(W.seeds(cfg, [(0.5 * nx * dx, 0.45 * ny * dx)], [1e17]))
    return cfgs, seeds


@pytest.mark.parametrize("kind", ["rect", "r4", "union", "union8"])
@pytest.mark.parametrize("least", ["0", "1000000000"])
def test_split_or_not_the_same_bits(kind, least, monkeypatch):
    """Groups always, where the surroundings leave room for them, and never;
    untuned stretches first."""
    cfgs, seeds = _batch(((384, 224), (320, 256)), kind)
    plain = [B.Sim(c, *s) for c, s in zip(cfgs, seeds)]
    monkeypatch.setenv("DMR_SPLIT_MIN", least)
    b = B.Batch(cfgs, seeds)
    for n in (40, 216, 256, 264, 504, 3):
        b.step(n)
        b.sync()
        for h, s in zip(b.instances, plain):
            s.step(n)
            assert h.patch() == s.patch()
            for lv in (0, 1):
                for f in FIELDS:
                    assert np.array_equal(h.get(f, lv), s.get(f, lv)), (n, f, lv)
    b.close()


def test_small_batches_take_the_step_in_one_launch():
    """One or a few small instances: the combined launch (10.8, 11.0, 11.5 us a
    step) is faster than a group's launches (14.2, 14.1, 14.5), and the tuner
    finds it.  Two of three, for what a timed choice is worth."""
    chosen = []
    for sizes in (((512, 256),), ((256, 128),), ((256, 128),) * 3):
        cfgs, seeds = _batch(sizes, field=1.2)
        b = B.Batch(cfgs, seeds)
        b.step(256)
        b.sync()
        chosen.append(b.config()[4])
        b.close()
    print(chosen)
    assert chosen.count("combined") >= 2

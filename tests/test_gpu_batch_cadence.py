"""A batch against plain runs where its own cadences (256-step intervals, the
steps it tunes on) and those of the run (growth tests, window blocks) do not
fall together."""
import numpy as np
import pytest

from paper_2105_13276_amd import binding as B
from paper_2105_13276_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("hz", "ex", "ey", "jx", "jy", "n", "acc", "ring")


def _same(h, s):
    for lv in (0, 1) if s.cfg["mode"] != "uniform" else (0,):
        for f in FIELDS:
            assert np.array_equal(h.get(f, lv), s.get(f, lv)), (f, lv)


def test_tuning_steps_over_no_growth_test():
    """First steps in calls too short to tune on; then a long call 32 steps
    before a growth test that grows the patch."""
    cfgs, seeds = [], []
    for side in (256, 384):
        cfg = W.make(side, side // 2, 32, "dynamic", 1, erms_over_ebd=4.0, regrid_every=800)
        dx = W.C0 / 110e9 / 32
        cfgs.append(cfg)
        seeds.append(W.seeds(cfg, [((side // 2 + 11.5) * dx, side // 4 * dx)], [3e17]))
    b = B.Batch(cfgs, seeds)
    plain = [B.Sim(c, *s) for c, s in zip(cfgs, seeds)]
    old = [s.patch() for s in plain]
    for n in (200, 200, 200, 168, 512, 300):
        b.step(n)
        b.sync()
        for h, s in zip(b.instances, plain):
            s.step(n)
            assert h.patch() == s.patch()
    assert any(s.patch() != o for s, o in zip(plain, old))
    for h, s in zip(b.instances, plain):
        _same(h, s)
    b.close()


@pytest.mark.parametrize("mode", ["uniform", "static"])
@pytest.mark.parametrize("cpl", [36, 128, 256])
def test_interval_that_holds_no_whole_periods(mode, cpl):
    """Window blocks of 9, 32 and 64 steps: 256 steps hold no whole number of
    them, one period, or half of one."""
    cfgs = [W.make(nx, 96, cpl, mode, 1, erms_over_ebd=2.0, tfsf_i=9,
                   static_ext=(nx // 2 - 8, 40, nx // 2 + 9, 57)) for nx in (96, 160)]
    g = np.random.Generator(np.random.PCG64(cpl))
    seeds = [(10.0 ** g.uniform(17, 20, (97, c["nx"] + 1)), None) for c in cfgs]
    b = B.Batch(cfgs, seeds)
    plain = [B.Sim(c, *s) for c, s in zip(cfgs, seeds)]
    for n in (1024, 256, 512):
        b.step(n)
        b.sync()
        for h, s in zip(b.instances, plain):
            s.step(n)
            _same(h, s)
    b.close()


def test_batches_tune_in_several_threads():
    """Batches that come to tune at the same time, in a thread each (the choices
    are kept for the whole process): the bits of the plain runs."""
    import threading
    cases, out = [], {}
    for k, nx in enumerate((160, 192, 224, 256)):
        cfg = W.make(nx, 96, 32, "dynamic", 1, erms_over_ebd=2.0)
        cases.append(([cfg, cfg], [W.seeds(cfg)] * 2))

    def run(k):
        import torch
        with torch.cuda.stream(torch.cuda.Stream()):
            b = B.Batch(*cases[k])
            for n in (256, 300, 44):
                b.step(n)
            b.sync()
            out[k] = [{f: h.get(f, 0) for f in FIELDS} for h in b.instances]
            b.close()

    threads = [threading.Thread(target=run, args=(k,)) for k in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k, (cfgs, seeds) in enumerate(cases):
        s = B.Sim(cfgs[0], *seeds[0])
        s.step(600)
        for got in out[k]:
            for f in FIELDS:
                assert np.array_equal(got[f], s.get(f, 0)), (k, f)
        s.close()

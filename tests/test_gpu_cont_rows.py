"""The base level's continuity with one, two and four rows a thread: the same
patch of density and window on a small grid (one row), on larger ones at every
row offset and against the top right corner, and in batches: the same bits."""
import numpy as np
import pytest

from paper_2105_13276_amd import binding as B
from paper_2105_13276_amd import workloads as W

pytestmark = pytest.mark.gpu

NX, NY, PAD, STEPS = 95, 60, 13, 12  # nodes 96 x 61; PAD > the steps' reach


def _small(corner):
    """Density and window values, random inside a frame of constant ones (none at
    the top and the right of the corner's)."""
    g = np.random.Generator(np.random.PCG64(5 + corner))
    inner = np.zeros((NY + 1, NX + 1), bool)
    inner[PAD:None if corner else -PAD, PAD:None if corner else -PAD] = True
    n = np.where(inner, 10.0 ** g.uniform(17, 20, inner.shape), 1e18)
    acc = [np.where(inner, (3e6 * g.uniform(0, 1, inner.shape)) ** 2, 0.0) for _ in range(STEPS)]
    return n, acc


def _cfg(nx, ny):
    # window blocks of one step; no field but the window values set below
    return W.make(nx, ny, 4, "uniform", 1, tfsf_i=0)


def _run(sims, step, n, acc):
    """n of every sim at the start; acc[k] before step k."""
    for s, a in zip(sims, n):
        B.Sim.set(s, "n", 0, a)
    for k in range(STEPS):
        for s, a in zip(sims, acc):
            B.Sim.set(s, "acc", 0, a[k])
        step()
    return [(s.get("n", 0), s.get("ring", 0)) for s in sims]


def _paste(nx, ny, small, places):
    n = np.full((ny + 1, nx + 1), 1e18)
    acc = [np.zeros((ny + 1, nx + 1)) for _ in range(STEPS)]
    for (j, i), (sn, sa) in zip(places, small):
        n[j:j + NY + 1, i:i + NX + 1] = sn
        for a, b in zip(acc, sa):
            a[j:j + NY + 1, i:i + NX + 1] = b
    return n, acc


@pytest.mark.parametrize("nx,ny", [(1040, 256), (2100, 2050), (4099, 1023)])
def test_rows_of_plain_runs(nx, ny):
    """Two rows a thread (267 K nodes) and four (4.3 and 4.2 M)."""
    one = [_small(0), _small(1)]
    ref = []
    for sn, sa in one:
        s = B.Sim(_cfg(NX, NY), None, None)
        ref += _run([s], lambda: s.step(1), [sn], [sa])
    places = [(63 * k, 1 + 200 * k) for k in range(4)] + [(ny - NY, nx - NX)]
    n, acc = _paste(nx, ny, [one[0]] * 4 + [one[1]], places)
    s = B.Sim(_cfg(nx, ny), None, None)
    got_n, got_r = _run([s], lambda: s.step(1), [n], [acc])[0]
    for (j, i), (rn, rr) in zip(places, [ref[0]] * 4 + [ref[1]]):
        assert np.array_equal(got_n[j:j + NY + 1, i:i + NX + 1], rn), (j, i)
        assert np.array_equal(got_r[:, j:j + NY + 1, i:i + NX + 1], rr), (j, i)
    assert (ref[0][0] != one[0][0].astype(np.float32)).any()


@pytest.mark.parametrize("count", [1, 7])
def test_rows_of_batches(count):
    """One row a thread (5.9 K nodes) and two (41 K)."""
    small = [_small(k & 1) for k in range(count)]
    b = B.Batch([_cfg(NX, NY)] * count, [(None, None)] * count)
    got = _run(b.instances, lambda: b.step(1), [q[0] for q in small], [q[1] for q in small])
    for k in range(count):
        s = B.Sim(_cfg(NX, NY), None, None)
        n, r = _run([s], lambda: s.step(1), [small[k][0]], [small[k][1]])[0]
        assert np.array_equal(got[k][0], n) and np.array_equal(got[k][1], r)
    b.close()

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

"""Workspace sizes (no device needed)."""
import pytest

from paper_2105_13276_amd import binding as B
from paper_2105_13276_amd import workloads as W


def _plane(nx, ny):
    return ((nx + 64) // 64 * 64 * (ny + 1) + 63) // 64 * 64 * 4


@pytest.mark.parametrize("kw,splits", [
    (dict(nx=512, ny=256, mode="dynamic"), False),
    (dict(nx=576, ny=448, mode="dynamic"), False),   # 2^18 cells less 4096
    (dict(nx=512, ny=512, mode="dynamic"), True),
    (dict(nx=512, ny=512, mode="dynamic", regrid_rule="union"), False),
    (dict(nx=1024, ny=512, mode="dynamic", regrid_rule="union"), True),
    (dict(nx=1024, ny=512, mode="dynamic", r=4), False),
    (dict(nx=1024, ny=1024, mode="dynamic", r=4), True),
    (dict(nx=1024, ny=512, mode="uniform"), False),
    # window blocks of 1 to 4 steps: groups as short pay on larger grids only
    (dict(nx=4096, ny=2048, mode="dynamic", cells_per_lambda=4), False),
    (dict(nx=1008, ny=1024, mode="dynamic", cells_per_lambda=8), False),
    (dict(nx=1024, ny=1024, mode="dynamic", cells_per_lambda=12), True),
    (dict(nx=512, ny=512, mode="dynamic", cells_per_lambda=16), True),
    (dict(nx=1024, ny=512, mode="dynamic", cells_per_lambda=8, regrid_rule="union"), False),
    (dict(nx=1024, ny=512, mode="dynamic", cells_per_lambda=12, regrid_rule="union"), True),
])
def test_third_set_of_planes_only_where_steps_are_split(kw, splits, monkeypatch):
    """The six planes (and for a union the map) of split steps are part of the
    size only where the grid can split."""
    cfg = W.make(periods=1, **dict(dict(cells_per_lambda=32), **kw))
    size = {}
    for least in (None, "0", "1000000000"):
        monkeypatch.delenv("DMR_SPLIT_MIN", raising=False)
        if least:
            monkeypatch.setenv("DMR_SPLIT_MIN", least)
        size[least] = B.workspace_bytes(cfg)
    assert size[None] == size["0" if splits else "1000000000"]
    if cfg["cells_per_lambda"] == 4:  # no group at all
        assert size["0"] == size[None]
        return
    more = 0 if cfg["mode"] == "uniform" else 6 * _plane(cfg["nx"], cfg["ny"])
    assert more <= size["0"] - size["1000000000"] <= more + (65536 if "regrid_rule" in kw else 0)

"""Kept children waiting for their chunks hold room for themselves, not for
every child of their batch: read from the library's trace lines (GV_TRACE),
with the results compared exactly (whole numbers) to the solve in one piece."""
import re
import sys

import numpy as np
import pytest

from paper_2107_11810_amd import synth

pytestmark = pytest.mark.gpu

LINE = re.compile(r"gv: level (\d+) cells (\d+) entries \d+ kept (\d+) \(room (\d+) of (\d+)\)")
SLACK = 65536  # children's room that is not worth a launch

PROBLEMS = {
    "plane3d": lambda: synth.plane3d(seed=7, n=400_003, n_in=4000, eps=(0.003, 0.003, 0.003)),
    "sim2d": lambda: synth.sim2d(seed=5, n_a=4000, k=9, n_in=500),
    "pose4dof": lambda: synth.pose4dof(seed=3, n=60_000, n_in=600),
}


@pytest.mark.parametrize("first_cells", ["", "3000"])  # parent order; several chunks in count order
@pytest.mark.parametrize("family", sorted(PROBLEMS))
def test_room_of_kept_children(monkeypatch, capfd, family, first_cells):
    from paper_2107_11810_amd import gvote
    g = PROBLEMS[family]()
    c = gvote.Context(0)
    try:
        ref = c.solve(g["family"], g["cols"], g["lo"], g["hi"], g["eps"])
        if first_cells:
            monkeypatch.setenv("GV_FIRST_CELLS", first_cells)
        monkeypatch.setenv("GV_TRACE", "1")
        capfd.readouterr()
        r = c.solve(g["family"], g["cols"], g["lo"], g["hi"], g["eps"])
        lines = [tuple(map(int, m.groups())) for m in LINE.finditer(capfd.readouterr().err)]
        monkeypatch.delenv("GV_TRACE")
    finally:
        c.close()
    print("kept room", family, first_cells, lines, flush=True)
    sys.stdout.flush()
    assert (r["count"], r["leaf_index"], r["sector"]) == (ref["count"], ref["leaf_index"], ref["sector"])
    assert np.array_equal(r["inliers"], ref["inliers"])
    assert any(kept and children - kept > SLACK for _, _, kept, _, children in lines), "no expansion that drops many"
    for _, _, kept, room, children in lines:
        assert kept == 0 or room - kept <= SLACK

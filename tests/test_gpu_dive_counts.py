"""The count pass that the dive leaves for the main search is taken by that
search's first batch only: solves whose dive goes greedy at every small
frontier size, with the look-ahead free to drop any child of it, equal the
oracle's (whole numbers)."""
import sys

import numpy as np
import pytest

import oracle
from paper_2107_11810_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2107_11810_amd import gvote
    c = gvote.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("probe", ["0", "2"])
@pytest.mark.parametrize("family", ["line2d", "plane3d", "ray3d", "sim2d", "pose4dof", "pose5dof"])
def test_greedy_from_any_frontier(ctx, monkeypatch, family, probe):
    monkeypatch.setenv("GV_PROBE", probe)
    g = synth.config(family + "_tiny")
    ro = oracle.solve(oracle.Problem(g["family"], g["cols"], g["lo"], g["hi"], g["eps"]))
    # around the cells of the levels where every axis splits, for one and for four root cells
    for cells in (2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 128, 256, 512, 1024):
        print("dive from", family, cells, "probe", probe, flush=True)
        sys.stdout.flush()
        monkeypatch.setenv("GV_DIVE_CELLS", str(cells))
        for group in (0, -1):
            r = ctx.solve(g["family"], g["cols"], g["lo"], g["hi"], g["eps"], group=group)
            assert (r["count"], r["leaf_index"], r["sector"]) == (ro["count"], ro["leaf_index"], ro["sector"])
            assert np.array_equal(r["inliers"], ro["inliers"])

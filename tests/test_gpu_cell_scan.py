"""Few long cells: a wave sums a (cell, child)'s items, 64 at a time.  Root
lists of just below, at and above 64 and 128 items of 256 entries, unit and
weighted, in lattice and exact mode.  Results equal those of items of 1024
entries, whose sums are one step of the wave (and which the oracle checks in
every other test), and for LINE2D the oracle's (whole numbers)."""
import math
import sys

import numpy as np
import pytest

import oracle
from paper_2107_11810_amd import synth

pytestmark = pytest.mark.gpu

MAKE = {
    "line2d": lambda n: synth.line2d(seed=n, n=n, n_in=n // 20),
    "plane3d": lambda n: synth.plane3d(seed=n, n=n, n_in=n // 20, sigma=0.004, eps=(0.04, 0.04, 0.04)),
    "sim2d": lambda n: synth.sim2d(seed=n, n_a=n, k=1, n_in=n // 10, sigma=0.003, eps=0.03),
    "pose4dof": lambda n: synth.pose4dof(seed=n, n=n, n_in=n // 30, noise_deg=0.2, eps_m=4.0, eps_deg=2.0,
                                         rho_max=80.0),
    "pose5dof": lambda n: synth.pose5dof(seed=n, n=n, n_in=n // 30, noise_deg=0.2, half_z=10.0, eps_m=4.0,
                                         eps_deg=2.0, eps_f_rel=0.05),
}


@pytest.fixture(scope="module")
def ctx():
    from paper_2107_11810_amd import gvote
    c = gvote.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", [64 * 256 - 1, 64 * 256, 64 * 256 + 1, 128 * 256 + 1])
@pytest.mark.parametrize("family", sorted(MAKE))
def test_items_of_long_cells(ctx, monkeypatch, family, n):
    g = MAKE[family](n)
    a = (g["family"], g["cols"], g["lo"], g["hi"], g["eps"])
    for canon_c in (0.0, math.inf):
        for group in (-1, 1):
            print("cell scan", family, n, canon_c, group, flush=True)
            sys.stdout.flush()
            rs = []
            for entries in ("256", "1024"):
                monkeypatch.setenv("GV_ITEM_ENTRIES", entries)
                rs.append(ctx.solve(*a, canon_c=canon_c, group=group))
            if family == "line2d":
                rs.append(oracle.solve(oracle.Problem(*a, canon_c=canon_c)))
            for r in rs[1:]:
                assert (r["count"], r["leaf_index"], r["sector"]) == (
                    rs[0]["count"], rs[0]["leaf_index"], rs[0]["sector"])
                assert np.array_equal(r["inliers"], rs[0]["inliers"])

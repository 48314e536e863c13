"""Frontier bookkeeping at the edges of its workgroups, and the pose families'
index lists: results equal the oracle's.  All comparisons are exact (counts,
leaf indices and inlier sets are whole numbers).
"""
import os
import sys

import numpy as np
import pytest

import oracle
from paper_2107_11810_amd import synth

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def OP(g):
    return oracle.Problem(g["family"], g["cols"], g["lo"], g["hi"], g["eps"])


@pytest.fixture(scope="module")
def ctx():
    from paper_2107_11810_amd import gvote
    c = gvote.Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def full_entries():
    """A context whose lists keep full entries at every level."""
    from paper_2107_11810_amd import gvote
    old = os.environ.get("GV_PACK")
    os.environ["GV_PACK"] = "0"
    try:
        c = gvote.Context(0)
    finally:
        if old is None:
            del os.environ["GV_PACK"]
        else:
            os.environ["GV_PACK"] = old
    yield c
    c.close()


# below, at and above one and four elements a thread of a 1024-thread
# workgroup, and the 256-thread workgroups that take over above that
@pytest.mark.parametrize("cells", [1, 255, 257, 1023, 1024, 1025, 4095, 4096, 4097])
def test_frontier_edges(ctx, monkeypatch, cells):
    """GV_DIVE_CELLS moves the frontier from which the dive goes greedy,
    GV_FIRST_CELLS the cells of an expansion's first chunk; the low threshold
    keeps more than 4096 children at several levels."""
    monkeypatch.setenv("GV_DIVE_CELLS", str(cells))
    monkeypatch.setenv("GV_FIRST_CELLS", str(cells))
    g = synth.line2d(seed=6, n=600, n_in=60)
    ro = oracle.solve(OP(g))
    _say("frontier", cells)
    r = ctx.solve(g["family"], g["cols"], g["lo"], g["hi"], g["eps"])
    assert (r["count"], r["leaf_index"], r["sector"]) == (ro["count"], ro["leaf_index"], ro["sector"])
    assert np.array_equal(r["inliers"], ro["inliers"])
    io, co = oracle.report(OP(g), ro["count"] // 4)
    assert len(io) > 2 * 4097
    ig, cg, _ = ctx.report(g["family"], g["cols"], g["lo"], g["hi"], g["eps"], ro["count"] // 4)
    assert np.array_equal(ig, io) and np.array_equal(cg, co)


@pytest.mark.parametrize("n", [63, 64, 65, 1023, 1025])
@pytest.mark.parametrize("family", ["pose4dof", "pose5dof"])
def test_index_lists_change_nothing(ctx, full_entries, family, n):
    """Lists below the root as indices of its records (the default) and as
    full entries, in both precisions, in one chunk and in many."""
    g = getattr(synth, family)(seed=n, n=n, n_in=max(10, n // 16))
    ro = oracle.solve(OP(g))
    for precision in (0, 1):
        for chunk in (None, "65536"):
            for name, c in (("index", ctx), ("full", full_entries)):
                _say(family, n, "precision", precision, "chunk bytes", chunk, name)
                if chunk:
                    os.environ["GV_CHUNK_BYTES"] = chunk
                try:
                    r = c.solve(g["family"], g["cols"], g["lo"], g["hi"], g["eps"], precision=precision)
                finally:
                    os.environ.pop("GV_CHUNK_BYTES", None)
                assert (r["count"], r["leaf_index"], r["sector"]) == (ro["count"], ro["leaf_index"], ro["sector"])
                assert np.array_equal(r["inliers"], ro["inliers"])

"""Chunks at the edges of one workgroup, and frontiers of more workgroups than add up each other's sums (over 2048 of
256 threads): cells' items, pruned children, greedy picks and re-cut chunks
with their prefixes scanned between the launches.  Results equal the oracle's
(whole numbers)."""
import re
import sys

import numpy as np
import pytest

import oracle
from paper_2107_11810_amd import synth

pytestmark = pytest.mark.gpu

CHUNK = re.compile(r"gv: level \d+ chunk (\d+)-(\d+) of \d+")
TRACE = re.compile(r"gv: level \d+ cells (\d+) entries \d+ kept (\d+) \(room \d+ of (\d+)\)")


def _problem():
    g = synth.line2d(seed=6, n=3000, n_in=60, eps=(0.0007, 0.0007))
    return g, oracle.Problem(g["family"], g["cols"], g["lo"], g["hi"], g["eps"])


@pytest.fixture(scope="module")
def ctx():
    from paper_2107_11810_amd import gvote
    c = gvote.Context(0)
    yield c
    c.close()


def _trace(capfd):
    return [tuple(map(int, m.groups())) for m in TRACE.finditer(capfd.readouterr().err)]


@pytest.mark.parametrize("first_cells", [1 << 30, 2_200_000])  # one chunk a level; re-cut chunks of 2149 workgroups
def test_report_of_a_large_frontier(ctx, monkeypatch, capfd, first_cells):
    g, P = _problem()
    tau = 4
    io, co = oracle.report(P, tau, cap=1 << 24)
    print("large frontier", first_cells, "leaves", len(io), flush=True)
    sys.stdout.flush()
    monkeypatch.setenv("GV_FIRST_CELLS", str(first_cells))
    monkeypatch.setenv("GV_TRACE", "1")
    capfd.readouterr()
    ig, cg, _ = ctx.report(g["family"], g["cols"], g["lo"], g["hi"], g["eps"], tau, cap=1 << 24)
    lines = _trace(capfd)
    print(lines, flush=True)
    assert max(cells for cells, _, _ in lines) > 2048 * 256      # k_items
    assert max(children for _, _, children in lines) > 2048 * 1024  # k_front
    assert max(kept for _, kept, _ in lines) > 2_200_000
    assert np.array_equal(ig, io) and np.array_equal(cg, co)


def test_greedy_dive_of_a_large_frontier(ctx, monkeypatch, capfd):
    g, P = _problem()
    ro = oracle.solve(P)
    monkeypatch.setenv("GV_DIVE_CELLS", "530000")
    monkeypatch.setenv("GV_FIRST_CELLS", str(1 << 30))
    monkeypatch.setenv("GV_TRACE", "1")
    capfd.readouterr()
    r = ctx.solve(g["family"], g["cols"], g["lo"], g["hi"], g["eps"])
    err = capfd.readouterr().err
    assert max(int(m) for m in re.findall(r"cells (\d+) entries \d+ kept .*\(dive\)", err)) > 2048 * 256  # k_pick
    assert (r["count"], r["leaf_index"]) == (ro["count"], ro["leaf_index"])
    assert np.array_equal(r["inliers"], ro["inliers"])


# around one and four elements a thread of a 1024-thread workgroup
@pytest.mark.parametrize("cells", [1023, 1024, 1025, 4095, 4096, 4097])
def test_chunks_at_the_edges_of_a_workgroup(ctx, monkeypatch, capfd, cells):
    g = synth.line2d(seed=6, n=600, n_in=60)
    P = oracle.Problem(g["family"], g["cols"], g["lo"], g["hi"], g["eps"])
    tau = oracle.solve(P)["count"] // 8
    io, co = oracle.report(P, tau)
    monkeypatch.setenv("GV_FIRST_CELLS", str(cells))
    monkeypatch.setenv("GV_TRACE", "1")
    print("chunk edges", cells, flush=True)
    sys.stdout.flush()
    capfd.readouterr()
    ig, cg, _ = ctx.report(g["family"], g["cols"], g["lo"], g["hi"], g["eps"], tau)
    sizes = [int(m[2]) - int(m[1]) for m in CHUNK.finditer(capfd.readouterr().err)]
    assert cells in sizes
    assert np.array_equal(ig, io) and np.array_equal(cg, co)

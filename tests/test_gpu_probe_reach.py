"""The look-ahead's tests reach what they are about: every kind of list it
reads, several chunks of one parent in parent and in count order, and children
it drops.  Seen in the library's trace lines (GV_TRACE); leaves and counts
equal the oracle's (whole numbers)."""
import os
import re
import sys

import numpy as np
import pytest

import oracle
from paper_2107_11810_amd import synth

pytestmark = pytest.mark.gpu

CHUNK = re.compile(r"gv: level \d+ chunk (\d+)-(\d+) of (\d+)( by count)?(?: probed (\w+))?: (\d+) left")

def _flat(n_in, n=2500):
    """Nearly level plane among points of all heights; slopes of a few steps
    beside heights of thousands, lists of the 8 | 8 | 16 word.  The planted
    share lies between the heights' parts of two levels, so that children
    pass whose own children do not."""
    rng = np.random.default_rng(77)
    x, y = rng.uniform(0.0, 1.0, n), rng.uniform(0.0, 1.0, n)
    z = rng.uniform(-2.0, 3.0, n)
    z[:n_in] = 0.7 + 0.01 * x[:n_in] - 0.005 * y[:n_in] + rng.normal(0.0, 0.002, n_in)
    return {"family": "plane3d", "cols": [x, y, z], "lo": [-0.02, -0.02, -2.0], "hi": [0.02, 0.02, 3.0],
            "eps": [0.003, 0.003, 0.01]}


# (lists stay unit weight: group = -1)
PROBLEMS = {
    # steeper slopes keep the 8-byte entry down to the leaves
    "EntP3p": (lambda: dict(synth.plane3d(seed=4001, n=4001, n_in=400, sigma=0.004), lo=[-8.0, -8.0, -8.0],
                            hi=[8.0, 8.0, 8.0], eps=[0.1, 0.1, 0.04]), 1),
    "EntP3v": (lambda: synth.plane3d(seed=4001, n=4001, n_in=400, sigma=0.004, eps=(0.04, 0.04, 0.04)), 1),
    "EntP3u": (lambda: _flat(430), 1),
    "EntI32": (lambda: synth.pose4dof(seed=5003, n=5003, n_in=300, noise_deg=0.2, eps_m=4.0, eps_deg=2.0,
                                      rho_max=80.0), 1),
    "EntI64": (lambda: synth.pose4dof(seed=5003, n=5003, n_in=300, noise_deg=0.2, eps_m=4.0, eps_deg=2.0,
                                      rho_max=80.0), 0),
    "EntI32 5": (lambda: synth.config("pose5dof_small"), 1),
    "EntI64 5": (lambda: synth.config("pose5dof_small"), 0),
}


@pytest.fixture(scope="module")
def ctx():
    from paper_2107_11810_amd import gvote
    c = gvote.Context(0)
    yield c
    c.close()


def _chunks(capfd):
    return [(int(m[1]), int(m[2]), int(m[3]), bool(m[4]), m[5], int(m[6]))
            for m in CHUNK.finditer(capfd.readouterr().err)]


@pytest.mark.parametrize("name", sorted(PROBLEMS))
def test_probe_of_every_list(ctx, monkeypatch, capfd, name):
    make, precision = PROBLEMS[name]
    g = make()
    a = (g["family"], g["cols"], g["lo"], g["hi"], g["eps"])
    ro = oracle.solve(oracle.Problem(*a))
    tau = 3 * ro["count"] // 4
    io, co = oracle.report(oracle.Problem(*a), tau)
    monkeypatch.setenv("GV_TRACE", "1")
    monkeypatch.setenv("GV_SUBTREE", "0")
    seen = {}
    for probe in ("0", "2"):
        for first in ("50", "400"):  # cells of a parent's first chunk
            monkeypatch.setenv("GV_PROBE", probe)
            monkeypatch.setenv("GV_FIRST_CELLS", first)
            print("probe reach", name, probe, first, flush=True)
            sys.stdout.flush()
            capfd.readouterr()
            r = ctx.solve(*a, precision=precision, group=-1)
            assert (r["count"], r["leaf_index"], r["sector"]) == (ro["count"], ro["leaf_index"], ro["sector"])
            assert np.array_equal(r["inliers"], ro["inliers"])
            ig, cg, _ = ctx.report(*a, tau, precision=precision, group=-1)
            assert np.array_equal(ig, io) and np.array_equal(cg, co)
            seen.setdefault(probe, []).extend(_chunks(capfd))
    entry = name.split()[0]
    assert not any(c[4] for c in seen["0"])
    probed = [c for c in seen["2"] if c[4] == entry]
    print(len(probed), "chunks probed,", sum(r1 - r0 - left for r0, r1, _, _, _, left in probed), "children dropped")
    assert any(left < r1 - r0 for r0, r1, _, _, _, left in probed)          # drops
    assert any(left > 0 for r0, r1, _, _, _, left in probed)                # and keeps
    assert any(r0 > 0 for r0, *_ in probed)                                 # later chunks of a parent
    assert any(by for _, _, _, by, _, _ in probed)                          # in count order

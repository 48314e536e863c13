"""A problem that fails in its root kernels (non-finite observation) beside
valid ones in one epoch: every valid problem's result is that of solving it
alone (whole numbers, compared exactly), wherever the failed one stands."""
import math
import os
import sys

import numpy as np
import pytest

from paper_2107_11810_amd import synth

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    """One serving lane, epochs shared by every problem that waits."""
    from paper_2107_11810_amd import gvote
    env = {"GV_BATCH_N": "1000000", "GV_LANES": "1"}
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    c = gvote.Context(0)
    for k, v in old.items():
        os.environ.pop(k) if v is None else os.environ.__setitem__(k, v)
    yield c
    c.close()


def same(a, b):
    return (a["count"] == b["count"] and a["leaf_index"] == b["leaf_index"] and a["sector"] == b["sector"]
            and np.array_equal(a["inliers"], b["inliers"]) and a["point"] == b["point"])


def problems(family, repeat):
    """Two valid problems and a failing one of one level structure; `repeat`
    copies of every observation, so that equal root surfaces merge."""
    make = {
        "line2d": lambda s: synth.line2d(seed=s, n=700, n_in=70),
        "plane3d": lambda s: synth.plane3d(seed=s, n=900, n_in=90, sigma=0.004, eps=(0.04, 0.04, 0.04)),
        "ray3d": lambda s: synth.ray3d(seed=s, n=900, n_in=90, noise_deg=0.2, eps=2.0),
        "sim2d": lambda s: synth.sim2d(seed=s, n_a=300, k=3, n_in=60, sigma=0.003, eps=0.03),
        "pose4dof": lambda s: synth.pose4dof(seed=s, n=900, n_in=90, noise_deg=0.2, eps_m=4.0, eps_deg=2.0,
                                             rho_max=80.0),
        "pose5dof": lambda s: synth.pose5dof(seed=s, n=600, n_in=60, noise_deg=0.2, half_z=10.0, eps_m=4.0,
                                             eps_deg=2.0, eps_f_rel=0.05),
    }[family]
    gs = [make(s) for s in (21, 22, 23)]
    for g in gs:
        g["cols"] = [np.repeat(np.asarray(c), repeat) for c in g["cols"]]
    gs[2]["cols"][0] = gs[2]["cols"][0].copy()
    gs[2]["cols"][0][5] = math.nan
    return gs


@pytest.mark.parametrize("order", [(2, 0), (2, 0, 1), (0, 2, 1), (0, 1, 2)])
@pytest.mark.parametrize("repeat", [1, 2])
@pytest.mark.parametrize("canon_c", [0.0, math.inf])
@pytest.mark.parametrize("family", ["line2d", "plane3d", "ray3d", "sim2d", "pose4dof", "pose5dof"])
def test_failed_problem_leaves_the_others_alone(ctx, family, canon_c, repeat, order):
    from paper_2107_11810_amd import gvote
    gs = problems(family, repeat)
    lo, hi, eps = gs[0]["lo"], gs[0]["hi"], gs[0]["eps"]
    _say("shared epoch", family, canon_c, repeat, order)
    ref = {i: ctx.solve(family, gs[i]["cols"], lo, hi, eps, canon_c=canon_c) for i in order if i != 2}
    # the lane is busy with the first problem while the rest queue up
    first = synth.pose4dof(seed=9, n=50_000, n_in=700)
    busy = gvote.submit(ctx, "pose4dof", first["cols"], first["lo"], first["hi"], first["eps"])
    tickets = [(i, gvote.submit(ctx, family, gs[i]["cols"], lo, hi, eps, canon_c=canon_c)) for i in order]
    assert gvote.poll(ctx, busy, 50_000)[0] == 0
    got = {}
    for i, t in tickets:
        st, r = gvote.poll(ctx, t, len(gs[i]["cols"][0]))
        assert st == (-1 if i == 2 else 0)
        got[i] = r
    for i, r in ref.items():
        assert same(got[i], r), i
    if len(ref) == 2:  # one epoch: its problems carry the same statistics
        assert got[0]["stats"]["ms_total"] == got[1]["stats"]["ms_total"]

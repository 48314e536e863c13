"""The device's range check of packed list entries answers on every call that
builds lists: with lists packed further up than the lattice bounds allow
(library knob GV_PACK_FROM, read when a call starts), a value that does not
fit ends in GV_ERANGE from gv_solve, gv_solve_noalloc and gv_report alike."""
import sys

import pytest

from paper_2107_11810_amd import synth

pytestmark = pytest.mark.gpu

# dependent axes fine enough that slopes at level 1 pass 32767 steps (4095 for
# PLANE3D), parameter axes coarse (not so coarse that millions of leaves tie)
PROBLEMS = {
    "line2d": lambda: synth.line2d(seed=1, n=200, n_in=40, sigma=2e-6, eps=(0.05, 1e-5)),
    "plane3d": lambda: synth.plane3d(seed=1, n=200, n_in=40, sigma=2e-5, eps=(0.05, 0.05, 1e-4)),
    "ray3d": lambda: synth.ray3d(seed=1, n=200, n_in=40, noise_deg=1e-4, eps=0.002),
    "sim2d": lambda: dict(synth.sim2d(seed=1, n_a=60, k=2, n_in=20, sigma=2e-5), eps=[0.01, 0.01, 1e-4, 1e-4]),
}


@pytest.fixture(scope="module")
def ctx():
    from paper_2107_11810_amd import gvote
    c = gvote.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("family", sorted(PROBLEMS))
def test_unpackable_value_is_refused(ctx, monkeypatch, family):
    from paper_2107_11810_amd import gvote
    g = PROBLEMS[family]()
    a = (g["family"], g["cols"], g["lo"], g["hi"], g["eps"])
    print("pack range", family, flush=True)
    sys.stdout.flush()
    best = ctx.solve(*a)
    leaves, counts, _ = ctx.report(*a, best["count"])
    assert best["leaf_index"] in leaves and (counts == best["count"]).all()
    monkeypatch.setenv("GV_PACK_FROM", "1")
    for call in (lambda: ctx.solve(*a), lambda: ctx.solve(*a, noalloc=True), lambda: ctx.report(*a, best["count"])):
        with pytest.raises(gvote.GvError) as e:
            call()
        assert e.value.status == -9
    monkeypatch.delenv("GV_PACK_FROM")
    assert ctx.report(*a, best["count"])[0].tolist() == leaves.tolist()

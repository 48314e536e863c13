"""Host waits that poll for their totals and host waits that only wait for the
stream (GV_POLL_US=0) give the same results on every call that makes them."""
import os
import sys

import numpy as np
import pytest

from paper_2107_11810_amd import synth

pytestmark = pytest.mark.gpu


def _context(poll_us):
    from paper_2107_11810_amd import gvote
    old = os.environ.get("GV_POLL_US")
    os.environ["GV_POLL_US"] = poll_us
    try:
        return gvote.Context(0)
    finally:
        os.environ.pop("GV_POLL_US") if old is None else os.environ.__setitem__("GV_POLL_US", old)


@pytest.fixture(scope="module")
def contexts():
    cs = [_context(us) for us in ("200", "0", "1")]
    yield cs
    for c in cs:
        c.close()


def same(a, b):
    return (a["count"] == b["count"] and a["leaf_index"] == b["leaf_index"] and a["sector"] == b["sector"]
            and np.array_equal(a["inliers"], b["inliers"]) and a["point"] == b["point"])


@pytest.mark.parametrize("family", ["line2d", "plane3d", "ray3d", "sim2d", "pose4dof", "pose5dof"])
def test_polled_or_waited_for(contexts, family):
    from paper_2107_11810_amd import gvote
    g = synth.config(family + ("_tiny" if family == "pose5dof" else "_small"))
    a = (g["family"], g["cols"], g["lo"], g["hi"], g["eps"])
    ref = contexts[0].solve(*a)
    rep = contexts[0].report(*a, ref["count"])
    for c in contexts[1:]:
        print("poll", family, flush=True)
        sys.stdout.flush()
        assert same(c.solve(*a), ref)
        assert same(c.solve(*a, noalloc=True), ref)
        leaves, counts, _ = c.report(*a, ref["count"])
        assert np.array_equal(leaves, rep[0]) and np.array_equal(counts, rep[1])
        st, r = gvote.poll(c, gvote.submit(c, *a), len(g["cols"][0]))
        assert st == 0 and same(r, ref)

"""The look-ahead takes a chunk by its rule only where its waves fill the chip
(a wave walks one list alone): small memory cuts chunks of a few cells, which
it must leave to the ordinary path.  Seen in the library's trace lines
(GV_TRACE); results equal those with memory for large chunks."""
import re
import sys

import numpy as np
import pytest

from paper_2107_11810_amd import synth

pytestmark = pytest.mark.gpu

CHUNK = re.compile(r"gv: level \d+ chunk (\d+)-(\d+) of \d+(?: by count)? probed \w+:")
SIMDS = 4 * 256  # of the chip: the fewest waves, and a chunk has at most a wave a child

PROBLEMS = {
    "plane3d": lambda: synth.plane3d(seed=1, n=120_000, n_in=3000, eps=(0.01, 0.01, 0.01)),
    "pose5dof": lambda: synth.pose5dof(seed=3, n=80_000, n_in=1300),
}


def _probed(capfd):
    return [int(m[2]) - int(m[1]) for m in CHUNK.finditer(capfd.readouterr().err)]


@pytest.mark.parametrize("name", sorted(PROBLEMS))
def test_small_chunks_are_not_probed(monkeypatch, capfd, name):
    from paper_2107_11810_amd import gvote
    monkeypatch.setenv("GV_TRACE", "1")
    g = PROBLEMS[name]()
    ctx, small = gvote.Context(0), gvote.Context(0, mem_budget_bytes=1 << 29)
    try:
        a = (g["family"], gvote.to_device(g["cols"]), g["lo"], g["hi"], g["eps"])
        got = []
        for which, c, noalloc in (("default", ctx, False), ("512 MiB", small, False), ("no allocation", ctx, True)):
            print("probe waves", name, which, flush=True)
            sys.stdout.flush()
            capfd.readouterr()
            r = c.solve(*a, noalloc=noalloc)
            sizes = _probed(capfd)
            print(len(sizes), "chunks probed, the smallest", min(sizes, default=None))
            assert min(sizes, default=SIMDS) >= SIMDS
            if which == "default":
                assert sizes  # (the rule still takes large chunks)
            got.append(r)
        for r in got[1:]:
            assert (r["count"], r["leaf_index"], r["sector"]) == tuple(got[0][k] for k in ("count", "leaf_index", "sector"))
            assert np.array_equal(r["inliers"], got[0]["inliers"])
    finally:
        ctx.close()
        small.close()

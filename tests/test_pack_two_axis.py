"""The packed list entries of RAY3D and SIM2D, on the host (exact round trips,
overflow flagged) and, on the GPU, against full entries and the oracle at
levels where every axis splits and where some no longer do."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2107_11810_amd import synth

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_two_axis_entries_round_trip(tmp_path):
    exe = str(tmp_path / "pack_two_axis")
    src = os.path.join(HERE, "host", "pack_two_axis_check.cpp")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-o", exe, src], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("OK")


def _uneven(g, factors):
    return dict(g, eps=[e * f for e, f in zip(g["eps"], factors)])


PROBLEMS = {
    "ray3d_1025": lambda: synth.ray3d(seed=1025, n=1025, n_in=120, noise_deg=0.2, eps=2.0),
    "ray3d_uneven": lambda: _uneven(synth.config("ray3d_small"), (1.0, 4.0, 2.0)),
    "sim2d_small": lambda: synth.config("sim2d_small", seed=61),
    "sim2d_uneven": lambda: _uneven(synth.config("sim2d_small"), (4.0, 1.0, 2.0, 1.0)),
    "line2d_uneven": lambda: _uneven(synth.config("line2d_small"), (1.0, 3.0)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(PROBLEMS))
@pytest.mark.parametrize("group", [0, 1])
def test_two_axis_packed_parity(name, group):
    from paper_2107_11810_amd import gvote
    g = PROBLEMS[name]()
    print("pack", name, group, flush=True)
    ro = oracle.solve(oracle.Problem(g["family"], g["cols"], g["lo"], g["hi"], g["eps"]))
    old = os.environ.get("GV_PACK")
    try:
        for pack in ("0", "1"):
            os.environ["GV_PACK"] = pack
            c = gvote.Context(0)
            try:
                r = c.solve(g["family"], g["cols"], g["lo"], g["hi"], g["eps"], group=group)
            finally:
                c.close()
            assert (r["count"], r["leaf_index"]) == (ro["count"], ro["leaf_index"]), pack
            assert np.array_equal(r["inliers"], ro["inliers"]), pack
    finally:
        if old is None:
            os.environ.pop("GV_PACK", None)
        else:
            os.environ["GV_PACK"] = old

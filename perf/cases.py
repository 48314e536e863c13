"""Timed cases of the voting library: what a caller has it do, from the smallest solve to the largest.

Every case is a plain dict; `prepare` makes the caller's inputs and keeps the library context that a program
holds, `run` makes one call (or, for serving, submits and polls one set of problems) and returns its results.
Inputs are the seeded planted-inlier data of paper_2107_11810_amd/synth.py at this repository's own
configurations and in between them.  Results are counts, leaves and inlier masks (whole numbers) and the returned
points; the library's timing statistics are not part of them.
"""
import math

import numpy as np
import torch

from paper_2107_11810_amd import gvote, synth

COLUMNS = {"line2d": 2, "plane3d": 3, "ray3d": 6, "sim2d": 4, "pose4dof": 5, "pose5dof": 5}
AXES = {"line2d": 2, "plane3d": 3, "ray3d": 3, "sim2d": 4, "pose4dof": 4, "pose5dof": 5}
SECTORS = {"pose4dof": 4, "pose5dof": 4}
# operations of one (surface, child box) test by the predicate's definition, children of a cell sharing terms
TEST_OPS = {"line2d": 6, "plane3d": 4, "ray3d": 12, "sim2d": 14, "pose4dof": 31, "pose5dof": 26}

_context = None


def context():
    """The one library context a program keeps (own stream, allocator and tuned launch shapes)."""
    global _context
    if _context is None:
        _context = gvote.Context(0)
    return _context


def _between(n, n0, v0, n1, v1):
    """The value at size n on the power law through (n0, v0) and (n1, v1)."""
    return v0 * (n / n0) ** (math.log(v1 / v0) / math.log(n1 / n0))


def _problem(case, seed):
    """The case's planted-inlier problem.  Inlier share, noise and eps follow the size between the
    repository's small and full-size configurations of each family."""
    family, n = case["family"], case["n"]
    if family == "line2d":
        inliers = max(3, round(n * _between(n, 2e3, 0.10, 1e4, 0.05))) if n < 10_000 else n // 20
        eps = max(0.005, _between(n, 2e3, 0.01, 1e4, 0.005))
        return synth.line2d(seed=seed, n=n, n_in=inliers, sigma=eps * 0.4, eps=(eps, eps))
    if family == "plane3d":
        eps = _between(n, 2e3, 0.04, 1e6, 0.003)
        inliers = round(n * _between(n, 2e3, 0.15, 1e6, 0.01))
        return synth.plane3d(seed=seed, n=n, n_in=inliers, sigma=_between(n, 2e3, 0.004, 1e6, 0.001),
                             eps=(eps, eps, eps))
    if family == "ray3d":
        return synth.ray3d(seed=seed, n=n, n_in=round(n * _between(n, 3e3, 0.10, 1e5, 0.01)),
                           noise_deg=_between(n, 3e3, 0.2, 1e5, 0.5), eps=_between(n, 3e3, 1.0, 1e5, 0.25))
    if family == "sim2d":
        points, k = n // case["candidates"], case["candidates"]
        return synth.sim2d(seed=seed, n_a=points, k=k, n_in=round(points * _between(points, 500, 0.16, 1e4, 0.10)),
                           sigma=_between(points, 500, 0.003, 1e4, 0.002), eps=_between(points, 500, 0.03, 1e4, 0.01))
    if family == "pose4dof":
        return synth.pose4dof(seed=seed, n=n, n_in=case["inliers"])
    return synth.pose5dof(seed=seed, n=n, n_in=round(n * _between(n, 3e3, 0.10, 2e4, 0.015)),
                          noise_deg=_between(n, 3e3, 0.2, 2e4, 0.5), half_z=_between(n, 3e3, 10.0, 2e4, 5.0),
                          eps_m=_between(n, 3e3, 4.0, 2e4, 0.5), eps_deg=_between(n, 3e3, 2.0, 2e4, 0.5),
                          eps_f_rel=_between(n, 3e3, 0.05, 2e4, 0.01))


def listed():
    return [
        # the smallest solve: 2,000 points still on the host; latency, launches and waits are all of it
        {"name": "line2d_2k_host", "call": "solve", "family": "line2d", "n": 2000, "host": True},
        # line fitting by duality at the paper's size
        {"name": "line2d_10k", "call": "solve", "family": "line2d", "n": 10_000, "host": False},
        # plane fitting on an ordinary scan, an odd number of points
        {"name": "plane3d_61k", "call": "solve", "family": "plane3d", "n": 61_003, "host": False},
        # plane fitting, the largest solve and the benchmark's default workload
        {"name": "plane3d_1m", "call": "solve", "family": "plane3d", "n": 1_000_000, "host": False},
        # camera position from rays with known orientation
        {"name": "ray3d_100k", "call": "solve", "family": "ray3d", "n": 100_000, "host": False},
        # every point that many rays meet (threshold reporting)
        {"name": "ray3d_report_20k", "call": "report", "family": "ray3d", "n": 20_011, "host": False},
        # similarity alignment: 10,000 points with nine candidate correspondences each
        {"name": "sim2d_90k", "call": "solve", "family": "sim2d", "n": 90_000, "candidates": 9, "host": False},
        # one query image's matches, every decision in binary64
        {"name": "pose4dof_50k_fp64", "call": "solve", "family": "pose4dof", "n": 50_021, "inliers": 700,
         "fp64": True, "host": False},
        # gravity-aligned pose against a whole model
        {"name": "pose4dof_1m", "call": "solve", "family": "pose4dof", "n": 1_000_000, "inliers": 5000,
         "fp64": False, "host": False},
        # pose with unknown focal length
        {"name": "pose5dof_20k", "call": "solve", "family": "pose5dof", "n": 20_000, "fp64": False, "host": False},
        # a serving process: problems of uneven size queued together and collected
        {"name": "serve_64", "call": "serve", "family": "pose4dof", "problems": 64},
        # verification and refinement of a vote's pose on its inlier set
        {"name": "refine_pose4dof", "call": "refine", "family": "pose4dof", "n": 200_000, "inliers": 4000},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["solve", "solve", "solve", "solve", "solve", "solve", "report", "serve", "refine"])
    if call == "serve":
        return {"call": "serve", "family": "pose4dof", "problems": rng.randint(5, 63), "mix": rng.randrange(100_000)}
    if call == "refine":
        n = _log_uniform(rng, 5_000, 400_000)
        return {"call": "refine", "family": "pose4dof", "n": n, "inliers": _log_uniform(rng, 100, min(5000, n // 10))}
    if call == "report":
        return {"call": "report", "family": "ray3d", "n": _log_uniform(rng, 3_000, 100_000), "host": False}
    family = rng.choice(["line2d", "plane3d", "ray3d", "sim2d", "pose4dof", "pose5dof"])
    case = {"call": "solve", "family": family, "host": rng.random() < 0.25}
    if family == "sim2d":
        case["candidates"] = rng.randint(6, 9)
        case["n"] = case["candidates"] * _log_uniform(rng, 500, 10_000)
    else:
        lo, hi = {"line2d": (2_000, 1_000_000), "plane3d": (2_000, 700_000), "ray3d": (3_000, 100_000),
                  "pose4dof": (1_000, 200_000), "pose5dof": (3_000, 20_000)}[family]
        case["n"] = _log_uniform(rng, lo, hi)
    if family in SECTORS:
        case["fp64"] = rng.random() < 0.3
    if family == "pose4dof":
        # the serving recipe's inlier shares; at least 30 inliers, so that the vote has a subject
        case["inliers"] = max(30, round(case["n"] * math.exp(rng.uniform(math.log(0.002), math.log(0.1)))))
    return case


def _columns(g, host):
    """Observation columns where the caller has them: binary64 vectors on the GPU, or host arrays."""
    return g["cols"] if host else [torch.from_numpy(c).cuda() for c in g["cols"]]


def _levels(g):
    """Leaf levels per axis: the smallest L with side * 2^-L <= eps (yaw: the tangent's [-1, 1])."""
    sides = [2.0 if j == 3 else g["hi"][j] - g["lo"][j] for j in range(len(g["eps"]))]
    levels = []
    for side, eps in zip(sides, g["eps"]):
        level = 0
        while math.ldexp(side, -level) > eps:
            level += 1
        levels.append(level)
    return sides, levels


def _truth_leaf(g):
    """The leaf holding the planted pose: (index, leaf-centre pose)."""
    x, y, z, yaw = g["truth"][:4]
    sector = int(math.floor((yaw + math.pi / 4) / (math.pi / 2))) % 4
    place = [x, y, z, math.tan(yaw - sector * math.pi / 2)]
    sides, levels = _levels(g)
    low = list(g["lo"][:3]) + [-1.0]
    cell = [min(max(int((p - a) / s * 2**L), 0), 2**L - 1) for p, a, s, L in zip(place, low, sides, levels)]
    index = sector
    for m in range(max(levels)):
        for c, L in zip(cell, levels):
            if m < L:
                index = (index << 1) | ((c >> (L - 1 - m)) & 1)
    centre = [a + s * (c + 0.5) / 2**L for a, s, c, L in zip(low, sides, cell, levels)]
    return index, centre[:3] + [sector * math.pi / 2 + math.atan(centre[3])]


REPORT_CAP = 16_384
REFINE = {"tau0": math.radians(1.5), "tau": math.radians(0.75), "rounds": 3, "iters": 10}


def _refine_inputs(case, seed):
    """A vote's leaf and inlier set: the planted matches with a few per cent of others among them."""
    g = _problem(case, seed)
    rng = np.random.default_rng(seed)
    others = np.setdiff1d(rng.integers(0, case["n"], size=case["inliers"] // 30 + 1), g["planted"])
    index, pose = _truth_leaf(g)
    return g, index, pose, np.sort(np.concatenate([g["planted"], others]))


def _serve_sizes(case):
    """The serving recipe: matches log-uniform in 1e3-2e5, inlier ratio log-uniform in 0.2%-10%."""
    rng = np.random.default_rng(case.get("mix", 199))
    sizes = np.exp(rng.uniform(math.log(1e3), math.log(2e5), size=case["problems"])).round().astype(int)
    ratios = np.exp(rng.uniform(math.log(0.002), math.log(0.1), size=case["problems"]))
    return [(int(n), max(3, round(n * r))) for n, r in zip(sizes, ratios)]


def prepare(case, seed):
    ctx = context()
    if case["call"] == "serve":
        gs = [synth.pose4dof(seed=100_000 * (seed % 20_000) + i, n=n, n_in=inliers)
              for i, (n, inliers) in enumerate(_serve_sizes(case))]
        state = {"problems": [(g, _columns(g, False)) for g in gs]}
    elif case["call"] == "refine":
        g, index, _, chosen = _refine_inputs(case, seed)
        state = {"g": g, "cols": _columns(g, False), "leaf": index, "idx": chosen}
    else:
        g = _problem(case, seed)
        state = {"g": g, "cols": _columns(g, case["host"]),
                 "precision": gvote.FP64_PLAIN if case.get("fp64") else gvote.FP32_FILTER}
        if case["call"] == "report":
            state["tau"] = max(8, len(g["planted"]) // 8)
    torch.cuda.synchronize()  # the library works on a stream of its own
    return {"ctx": ctx, "call": case["call"], **state}


def _mask(n, chosen):
    """The chosen observations as a caller uses them: one flag each."""
    m = np.zeros(n, dtype=bool)
    m[chosen] = True
    return m


def _result(r, n):
    return {"count": r["count"], "leaf": r["leaf_index"], "sector": r["sector"], "coords": np.array(r["leaf_coords"]),
            "point": np.array(r["point"]), "bound": np.array(r["bound"]), "inliers": _mask(n, r["inliers"])}


def run(state):
    ctx = state["ctx"]
    if state["call"] == "serve":
        tickets = [gvote.submit(ctx, g["family"], cols, g["lo"], g["hi"], g["eps"]) for g, cols in state["problems"]]
        done = []
        for ticket, (g, _) in zip(tickets, state["problems"]):
            status, r = gvote.poll(ctx, ticket, len(g["cols"][0]))
            if status != 0:
                raise RuntimeError(f"poll: status {status}")
            done.append(r)
        return {"counts": np.array([r["count"] for r in done]), "leaves": np.array([r["leaf_index"] for r in done]),
                "points": np.array([r["point"] for r in done]),
                "inliers": np.concatenate([_mask(len(g["cols"][0]), r["inliers"])
                                           for r, (g, _) in zip(done, state["problems"])])}
    g = state["g"]
    n = len(g["cols"][0])
    where = (g["family"], state["cols"], g["lo"], g["hi"], g["eps"])
    if state["call"] == "refine":
        r = ctx.refine(*where, state["leaf"], state["idx"], **REFINE)
        return {**r, "verified": _mask(n, r["verified"])}
    if state["call"] == "report":
        leaves, counts, _ = ctx.report(*where, state["tau"], cap=REPORT_CAP, precision=state["precision"])
        out = np.zeros((2, REPORT_CAP), dtype=np.int64)  # zeros behind the last leaf
        out[0, :len(leaves)], out[1, :len(leaves)] = leaves, counts
        return {"leaves": out[0], "counts": out[1]}
    return _result(ctx.solve(*where, precision=state["precision"]), n)


def _size(family, n):
    """Every observation is read once, parametrized, and tested against the children of the root."""
    children = 2 ** AXES[family] * SECTORS.get(family, 1)
    return 8.0 * COLUMNS[family] * n, float(n * children * TEST_OPS[family])


def work(case):
    if case["call"] == "serve":
        moved, ops = _size("pose4dof", sum(n for n, _ in _serve_sizes(case)))
    elif case["call"] == "refine":
        # 3 rounds of 10 steps: about 200 operations a match and step for residual, Jacobian and sums
        n = case["inliers"]
        moved, ops = 8.0 * (COLUMNS["pose4dof"] + 2) * n, 200.0 * 30 * n
    else:
        moved, ops = _size(case["family"], case["n"])
    return {"bytes": moved, "flops": ops}


def _directions(q, w, xi, eta):
    """Unit observed and predicted directions (camera axes: forward, lateral, up), distance and d."""
    o = np.stack([np.ones_like(xi), xi, eta * np.sqrt(1.0 + xi * xi)], axis=1)
    d = w - np.asarray(q[:3])[None, :]
    c, s = math.cos(q[3]), math.sin(q[3])
    d = np.stack([c * d[:, 0] + s * d[:, 1], c * d[:, 1] - s * d[:, 0], d[:, 2]], axis=1)
    far = np.linalg.norm(d, axis=1, keepdims=True)
    return o / np.linalg.norm(o, axis=1, keepdims=True), d / far, far, d


def _kept(q, w, xi, eta, tau):
    o, u, _, _ = _directions(q, w, xi, eta)
    return np.arctan2(np.linalg.norm(np.cross(o, u), axis=1), np.sum(o * u, axis=1)) <= tau


def _rms(q, w, xi, eta):
    o, u, _, _ = _directions(q, w, xi, eta)
    return math.sqrt(np.mean(np.sum((u - o) ** 2, axis=1))) if len(o) else 0.0


def exact(case, seed):
    """Refinement: the least-squares pose on the verified matches, in numpy.  The other calls' floating
    outputs are leaf centres and bounds of a search that has no short form."""
    if case["call"] != "refine":
        return None
    g, _, q, chosen = _refine_inputs(case, seed)
    X = [c[chosen] for c in g["cols"]]
    w, xi, eta = np.stack(X[:3], axis=1), X[3], X[4]
    keep = _kept(q, w, xi, eta, REFINE["tau0"])
    rms0 = _rms(q, w[keep], xi[keep], eta[keep])
    q = np.array(q)
    for _ in range(REFINE["rounds"]):
        for _ in range(REFINE["iters"]):
            o, u, far, d = _directions(q, w[keep], xi[keep], eta[keep])
            c, s = math.cos(q[3]), math.sin(q[3])
            turn = np.stack([d[:, 1], -d[:, 0], 0 * d[:, 2]], axis=1)
            cols = [np.broadcast_to(v, d.shape) for v in ([-c, s, 0.0], [-s, -c, 0.0], [0.0, 0.0, -1.0])] + [turn]
            J = np.stack([(v - u * np.sum(u * v, axis=1, keepdims=True)) / far for v in cols], axis=2).reshape(-1, 4)
            q = q + np.linalg.lstsq(J, -(u - o).reshape(-1), rcond=None)[0]
        keep = _kept(q, w, xi, eta, REFINE["tau"])
    pose = np.append(q, 0.0)
    pose[3] %= 2 * math.pi
    return {"pose": list(pose), "rms": _rms(q, w[keep], xi[keep], eta[keep]), "rms0": rms0,
            "verified": _mask(case["n"], chosen[keep])}

"""Iterations replayed from captured HIP graphs against the same launches issued one by one, bit for bit, on sets that
are captured (more than 64 edges, or more than 128 unknowns): dense features with split spread passes, class ids, a
block-sparse solve.  Every case replays over repeated calls, with eager work between them, and after a rebuild; that
graphs were launched at all is read from the runtime's log of a process of its own."""
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
from helpers import ROOT

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]

N_ITER = 4


def make(kind, seed):
    """Clouds, features, poses and edges of a set that is captured."""
    rng = np.random.default_rng(seed)
    K = {"dense": 12, "bf16": 12, "class": 12, "chain": 30}[kind]
    n = 700
    base = rng.uniform(0.0, 1.2, size=(n, 3))
    base[::3] = rng.uniform(0.0, 12.0, size=(len(base[::3]), 3))  # scattered points: spread passes of many rows
    pts, poses = [], []
    for k in range(K):
        T = oracle.se3_exp(rng.normal(scale=0.01, size=6))
        R, t = T[:9].reshape(3, 3), T[9:]
        pts.append(((base + rng.normal(scale=0.02, size=base.shape) - t) @ R).astype(np.float32))
        poses.append(oracle.se3_exp(rng.normal(scale=0.01, size=6)))
    if kind in ("class", "chain"):
        ids = rng.integers(0, 4, size=n).astype(np.uint16)
        feats, feat = [ids] * K, "class"
    else:
        feats, feat = [rng.uniform(0.1, 1.0, size=(n, 9)).astype(np.float32) for _ in range(K)], kind
    edges = [(m, k) for m in range(K) for k in range(m + 1, K) if kind != "chain" or k - m <= 3]
    return pts, feats, feat, np.stack(poses), edges


def solve(ctx, kind, seed):
    pts, feats, feat, poses, edges = make(kind, seed)
    ctx.build_neighbors(pts, feats, feat)
    return poses, edges


@pytest.mark.parametrize("kind", ["dense", "bf16", "class", "chain"])
def test_replayed_iterations_are_the_launched_ones(kind):
    from paper_2403_01254_amd import rkhsba
    options = dict(ell=0.1, cell_subdiv=6, pass_points=16)
    with rkhsba.Context(use_graphs=True, **options) as g, rkhsba.Context(use_graphs=False, **options) as e:
        for seed in (1, 2):  # the second is a rebuild
            poses, edges = solve(g, kind, seed)
            solve(e, kind, seed)
            want = e.gn_step(poses, edges, N_ITER)
            assert want[2][0] > 0 and np.abs(want[0] - poses).max() > 1e-4
            for _ in range(3):
                got = g.gn_step(poses, edges, N_ITER)
                for x, y in zip(got, want):
                    np.testing.assert_array_equal(x, y)
                g.eval_loss(poses, edges[:5])
                g.accumulate_normal_eqs(poses, edges[::-1])
                moved = g.gn_step(got[0], edges, 2)  # replays from other poses
                for x, y in zip(moved, e.gn_step(want[0], edges, 2)):
                    np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("kind", ["dense", "class", "chain"])
def test_graphs_are_launched(kind):
    code = ("import sys; sys.path[:0] = [%r, %r]\n"
            "from paper_2403_01254_amd import rkhsba\n"
            "from test_gpu_graph_replay import N_ITER, solve\n"
            "with rkhsba.Context(ell=0.1, use_graphs=True) as c:\n"
            "    p, e = solve(c, %r, 1)\n"
            "    c.gn_step(p, e, N_ITER)\n" % (ROOT, os.path.join(ROOT, "tests"), kind))
    run = subprocess.run([sys.executable, "-c", code], check=True, capture_output=True, text=True, timeout=100,
                         env=dict(os.environ, AMD_LOG_LEVEL="3", AMD_LOG_MASK="1"))
    launches = [line for line in run.stderr.splitlines() if "hipGraphLaunch" in line and "(" in line]
    assert len(launches) >= N_ITER

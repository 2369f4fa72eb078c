"""Per-point walks where their loops turn: more cell rows than one round of ranges holds (12), ranges from one point to
many steps of four candidates, and, with top-k selection, exact ties of the kernel value (points on a grid),
candidates whose kernel value is 30 orders of magnitude below the kept ones', and fewer candidates than k; against the FP64 oracle and its selection."""
import numpy as np
import pytest

import oracle
from helpers import REL_TOL, assert_blocks_close, ident

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]

EDGES = [(0, 1), (1, 0)]


def clouds(rng, shape, n):
    if shape == "grid":
        pts = [rng.integers(-4, 5, size=(n, 3)) / 16.0 for _ in range(2)]
    elif shape == "columns":  # many points in few cells, and many empty rows between
        pts = [np.c_[rng.uniform(-0.5, 0.5, n), rng.choice([-0.4, 0.0, 0.35], n), rng.choice([-0.3, 0.3], n)]
               for _ in range(2)]
    else:
        pts = [rng.uniform(-0.5, 0.5, size=(n, 3)) for _ in range(2)]
    return [p.astype(np.float32) for p in pts]


def features(rng, feat, n):
    if feat == "class":
        return [rng.integers(0, 2, size=n).astype(np.uint16) for _ in range(2)]
    return [(rng.integers(1, 5, size=(n, 6)) / 4.0).astype(np.float32) for _ in range(2)]


@pytest.mark.parametrize("top_k", [0, 1, 3, 8])
@pytest.mark.parametrize("feat", ["class", "dense"])
@pytest.mark.parametrize("shape,n,subdiv,ell,cutoff", [
    ("uniform", 3, 1, 0.1, 3.0), ("uniform", 500, 1, 0.1, 3.0), ("uniform", 500, 4, 0.1, 3.0),
    ("uniform", 500, 8, 0.1, 3.0), ("columns", 700, 1, 0.1, 3.0), ("columns", 700, 8, 0.1, 3.0),
    ("grid", 400, 1, 0.1, 3.0), ("grid", 400, 3, 0.05, 3.0), ("uniform", 1500, 1, 0.03, 12.0)])
def test_walks(shape, n, subdiv, ell, cutoff, feat, top_k):
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(n + subdiv)
    pts, feats = clouds(rng, shape, n), features(rng, feat, n)
    poses = np.stack([ident(), ident()])
    if shape != "grid":
        poses[1, 9:] = [0.02, -0.01, 0.015]
    op = oracle.Problem(pts, feats, feat, ell, cutoff_factor=cutoff, top_k=top_k)
    oF, ob, oH, _, onp = oracle.normal_eqs(op, poses, EDGES, oracle.MEMBER_FP32_RULE)
    with rkhsba.Context(ell=ell, cutoff_factor=cutoff, top_k=top_k, cell_subdiv=subdiv, pass_points=1) as ctx:
        ctx.build_neighbors(pts, feats, feat)
        H, b, F, n_pairs = ctx.accumulate_normal_eqs(poses, EDGES)
        lF, _, l_pairs = ctx.eval_loss(poses, EDGES)
        if top_k:
            np.testing.assert_array_equal(ctx.export_pairs(poses, 0, 1), oracle.pairs(op, poses, 0, 1))
    assert n_pairs == onp and l_pairs == onp
    assert abs(F - oF) <= REL_TOL * abs(oF) and abs(lF - oF) <= REL_TOL * abs(oF)
    assert_blocks_close(b, ob, 6, rel=REL_TOL, what="b")
    assert_blocks_close(H, oH, 6, rel=REL_TOL, what="H")

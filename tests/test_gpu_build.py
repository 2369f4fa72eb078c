"""Frame bounds, row tables and the cell-size choice of a build at the sizes where their kernels change course: frames
around a chunk of 1,024 points and of unequal sizes, negative coordinates, row tables around 32,768 rows (one workgroup
up to there) and a grid that is built again after the occupancy is known.  The reported occupancy is NumPy's count of
occupied cells; losses and pair counts are the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from helpers import REL_TOL, ident

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]


def occupancy(pts, ids, r_c):
    cells = 0
    for p, l in zip(pts, ids):
        k = np.floor(p.astype(np.float64) * (1.0 / r_c)).astype(np.int64)
        cells += len(np.unique(np.c_[k, l], axis=0))
    return sum(len(p) for p in pts) / cells


def evaluate(rkhsba, pts, feats, feat, ell, **options):
    poses = np.stack([ident() for _ in pts])
    poses[1, 9:] = [0.03, -0.02, 0.01]
    edges = [(0, 1), (1, 0)]
    op = oracle.Problem(pts, feats, feat, ell)
    oF, _, _, _, onp = oracle.normal_eqs(op, poses, edges, oracle.MEMBER_FP32_RULE)
    with rkhsba.Context(ell=ell, **options) as ctx:
        ctx.build_neighbors(pts, feats, feat)
        F, _, n = ctx.eval_loss(poses, edges)
        config = ctx.config()
    assert n == onp and abs(F - oF) <= REL_TOL * abs(oF)
    return config


@pytest.mark.parametrize("feat", ["class", "dense"])
@pytest.mark.parametrize("sizes", [(1, 1), (1, 3000), (1023, 1024), (1025, 7), (5000, 2), (300, 200, 17, 4097)])
def test_frames_of_any_size(feat, sizes):
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(sum(sizes))
    ell = 0.2
    pts = [rng.uniform(-1.0, 0.4, size=(n, 3)).astype(np.float32) for n in sizes]
    pts[1][0] = pts[0][0]  # a pair in any case
    if feat == "class":
        feats = [rng.integers(0, 5, size=n).astype(np.uint16) for n in sizes]
        feats[1][0] = feats[0][0]
    else:
        feats = [rng.uniform(0.1, 1.0, size=(n, 5)).astype(np.float32) for n in sizes]
    ids = feats if feat == "class" else [np.zeros(n, int) for n in sizes]
    want = occupancy(pts, ids, 3.0 * ell)
    assert evaluate(rkhsba, pts, feats, feat, ell)[2] == pytest.approx(want, rel=1e-12)
    assert evaluate(rkhsba, pts, feats, feat, ell, cell_subdiv=3)[0] == 3


# rows: cells along y times cells along z, of both frames; 2 x 128 x 128 = 32,768
@pytest.mark.parametrize("ny,nz", [(1, 1), (1, 512), (1, 513), (33, 31), (127, 129), (128, 128), (129, 128), (257, 256)])
def test_row_tables(ny, nz):
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(ny * nz)
    ell = 0.1
    r_c = 3.0 * ell
    n = 6000
    corner = np.array([[0.5, 0.5, 0.5], [7.5, ny - 0.5, nz - 0.5]])
    p = np.r_[corner, rng.uniform(0.0, 1.0, size=(n, 3)) * [8, ny, nz]] * r_c
    moved = np.clip(p + rng.normal(scale=0.02, size=p.shape), 1e-3, np.array([8, ny, nz]) * r_c - 1e-3)
    pts = [p.astype(np.float32), moved.astype(np.float32)]
    feats = [rng.uniform(0.1, 1.0, size=(len(q), 3)).astype(np.float32) for q in pts]
    evaluate(rkhsba, pts, feats, "dense", ell, cell_subdiv=1, pass_points=16)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf, 3e30])
@pytest.mark.parametrize("where", [0, 1024, 2999])
def test_refused_coordinates(value, where):
    from paper_2403_01254_amd import rkhsba
    pts = np.random.default_rng(0).uniform(size=(3000, 3)).astype(np.float32)
    pts[where, where % 3] = value
    ids = np.zeros(3000, np.uint16)
    with rkhsba.Context(ell=0.1) as ctx:
        for device in (False, True):
            p = torch.from_numpy(pts).cuda() if device else pts
            f = torch.from_numpy(ids.astype(np.int16)).cuda() if device else ids
            with pytest.raises(rkhsba.RkhsbaError) as err:
                ctx.build_neighbors([p, p], [f, f], "class")
            assert err.value.code == rkhsba.EINVAL

"""Sweep passes whose box spans many cell rows (their sources lie in a few places far apart), on both sides of the
limits from which row batches that no source is near are skipped and from which a pass is split over its sources
(whole quads, single sources, and more items than the list holds).  Per-source counts are the oracle's; the sums are
checked against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from helpers import REL_TOL, assert_blocks_close, ident

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]


def clusters(rng, centres, n, size):
    c = np.asarray(centres, dtype=np.float64)
    return (c[rng.integers(0, len(c), size=n)] + rng.uniform(-size, size, size=(n, 3))).astype(np.float32)


def check(rkhsba, pts, feats, feat, subdiv, ell, poses):
    edges = [(0, 1), (1, 0)]
    op = oracle.Problem(pts, feats, "dense", ell)
    with rkhsba.Context(ell=ell, cell_subdiv=subdiv, pass_points=16) as ctx:
        ctx.build_neighbors(pts, feats, feat)
        for m, n in edges:
            ref = oracle.pairs(op, poses, m, n)
            # of the pairs inside the radius, those with c > 0 (negative inner products are clamped to 0)
            c = np.sum(feats[m][ref[:, 0]].astype(np.float64) * feats[n][ref[:, 1]], axis=1)
            ref = ref[c > 0]
            assert len(ref) > 0
            np.testing.assert_array_equal(ctx.export_source_counts(poses, m, n, len(pts[m])),
                                          np.bincount(ref[:, 0], minlength=len(pts[m])))
        oF, ob, oH, _, onp = oracle.normal_eqs(op, poses, edges, oracle.MEMBER_FP32_RULE)
        H, b, F, n_pairs = ctx.accumulate_normal_eqs(poses, edges)
        lF, _, l_pairs = ctx.eval_loss(poses, edges)
        # fp8 products accumulate inexactly on the matrix cores (2.5e-4 elsewhere in these tests)
        tol = 2.5e-4 if feat == "fp8" else REL_TOL
        assert n_pairs == onp and l_pairs == onp
        assert abs(F - oF) <= tol * abs(oF) and abs(lF - oF) <= tol * abs(oF)
        assert_blocks_close(b, ob, 6, rel=tol, what="b")
        assert_blocks_close(H, oH, 6, rel=tol, what="H")


# extent of the clusters' placement in r_c: rows of a spread pass from below 512 to some 1e5 (more than 64 batches
# of 64 rows), cluster sizes from single points to several cells
@pytest.mark.parametrize("extent", [1.5, 3.0, 12.0, 40.0])
@pytest.mark.parametrize("feat", ["dense", "bf16", "fp8"])
@pytest.mark.parametrize("subdiv", [1, 8])
def test_spread_passes(feat, subdiv, extent):
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(int(10 * extent) + subdiv)
    ell = 0.1
    centres = rng.uniform(0.0, extent * 0.3, size=(7, 3))
    pts = [clusters(rng, centres, n, 0.05) for n in (500, 333)]
    # values that bfloat16 and fp8 store exactly
    feats = [(rng.integers(1, 9, size=(len(p), 9)) / 8.0).astype(np.float32) for p in pts]
    poses = np.stack([ident(), ident()])
    poses[1, 9:] = [0.02, -0.03, 0.01]
    check(rkhsba, pts, feats, feat, subdiv, ell, poses)


@pytest.mark.parametrize("dim", [5, 16, 20, 31, 64])
def test_scattered_sources(dim):
    """Every source far from the others: passes of 16 single-source items, several times what the list holds; every
    padded width of FP32 features."""
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(dim)
    x = rng.uniform(0.0, 18.0, size=(999, 3))
    pts = [x.astype(np.float32), (x + rng.uniform(-0.1, 0.1, size=x.shape)).astype(np.float32)]
    feats = [rng.normal(size=(len(p), dim)).astype(np.float32) for p in pts]  # both signs: clamped products
    check(rkhsba, pts, feats, "dense", 3, 0.1, np.stack([ident(), ident()]))

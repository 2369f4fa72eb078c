"""Voxel and binning sorts at the sizes where their route changes: one run of 2,048 elements in LDS, runs and
a merge (up to 16,384 elements), tiles with fused histogram sums (up to 64 tiles of 2,048), tiles with scanned
histograms.  Cell keys and their stable order are compared with the oracle's bit for bit; a binning that lost
or repeated a source point would change the per-source pair counts."""
import numpy as np
import pytest

import oracle
from helpers import ident, inv_cell

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]

EDGES = [1, 64, 65, 2048, 2049, 8192, 8193, 16384, 16385, 131072, 131073]


def cloud(rng, n):
    return rng.uniform(-3.0, 3.0, size=(n, 3)).astype(np.float32)


@pytest.mark.parametrize("kind", ["class", "dense"])
@pytest.mark.parametrize("n", EDGES)
def test_sort_routes(n, kind):
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(n)
    pts = [cloud(rng, n), cloud(rng, 300)]
    # class ids: label layers split the binning into segments of unequal sizes, a few of them empty
    lab = [rng.choice([0, 1, 5], p=[0.7, 0.2, 0.1], size=len(p)).astype(np.uint16) for p in pts]
    feats = lab if kind == "class" else [rng.uniform(0.1, 1.0, size=(len(p), 5)).astype(np.float32) for p in pts]
    ell, subdiv = 0.1, 3
    poses = np.stack([ident(), ident()])
    op = oracle.Problem(pts, feats, kind, ell)
    with rkhsba.Context(ell=ell, cell_subdiv=subdiv, pass_points=16) as ctx:
        ctx.build_neighbors(pts, feats, kind)
        for f in range(2):
            perm, keys, _, dims, layers = ctx.export_voxels(f, len(pts[f]))
            operm, okeys, _, odims = oracle.voxels(pts[f], inv_cell(ell, 3.0, subdiv),
                                                   labels=lab[f] if layers else None)
            np.testing.assert_array_equal(dims, odims)
            np.testing.assert_array_equal(keys, okeys)
            np.testing.assert_array_equal(perm, operm)
        for m, k in ((0, 1), (1, 0)):
            ref = oracle.pairs(op, poses, m, k)
            got = ctx.export_source_counts(poses, m, k, len(pts[m]))
            np.testing.assert_array_equal(got, np.bincount(ref[:, 0], minlength=len(pts[m])))


def test_mixed_routes_in_one_set():
    """Frames of every route in one problem (odd digit count: the sorts end in the second buffer)."""
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(0)
    sizes = [40000, 3, 2049, 140000, 9000, 500]
    pts = [cloud(rng, n) for n in sizes]
    feats = [rng.integers(0, 3, size=n).astype(np.uint16) for n in sizes]
    poses = np.stack([ident()] * len(sizes))
    op = oracle.Problem(pts, feats, "class", 0.02)
    for subdiv in (1, 8):
        with rkhsba.Context(ell=0.02, cell_subdiv=subdiv, pass_points=16) as ctx:
            ctx.build_neighbors(pts, feats, "class")
            edges = [(i, 5) for i in range(5)] + [(5, 3)]
            for i, j in edges:
                ref = oracle.pairs(op, poses, i, j)
                got = ctx.export_source_counts(poses, i, j, sizes[i])
                np.testing.assert_array_equal(got, np.bincount(ref[:, 0], minlength=sizes[i]))
            _, _, n_pairs = ctx.eval_loss(poses, edges)
            assert n_pairs == sum(len(oracle.pairs(op, poses, i, j)) for i, j in edges)

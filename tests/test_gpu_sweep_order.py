"""The order in which a dense sweep's workgroups take split passes' items and whole passes, on both sides of its limit
of 2,048 items in front: every item and every pass is taken once.  The allocation-free evaluation, which splits no
pass, gives the same F and pair counts, bit for bit."""
import numpy as np
import pytest

from helpers import ident

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]


def check(sizes, edges, spread, feat="dense"):
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(sum(sizes))
    x = rng.uniform(0.0, 40.0 if spread else 3.0, size=(max(sizes), 3))
    if spread == "half":
        x[:len(x) // 2] *= 0.05
    pts = [(x[:n] + rng.uniform(-0.1, 0.1, size=(n, 3))).astype(np.float32) for n in sizes]
    feats = [rng.uniform(0.1, 1.0, size=(n, 4)).astype(np.float32) for n in sizes]
    poses = np.stack([ident()] * len(sizes))
    with rkhsba.Context(ell=0.1, cell_subdiv=3, pass_points=16) as ctx:
        ctx.build_neighbors(pts, feats, feat)
        F, Fe, n = ctx.eval_loss(poses, edges)
        whole = ctx.eval_loss_noalloc(poses, edges)
    assert n > 0 and n == whole[2]
    np.testing.assert_array_equal(Fe, whole[1])


# passes of the set: 50, 1,938 (fewer items than the limit), 2,050 and 4,375 (a full list is above it)
@pytest.mark.parametrize("n", [800, 31000, 32800, 70000])
@pytest.mark.parametrize("spread", [False, "half", True])
def test_items_and_passes(n, spread):
    check((n, 3000), [(0, 1)], spread)


@pytest.mark.parametrize("feat", ["bf16", "fp8"])
def test_items_of_many_edges(feat):
    check((9001, 6000, 4000), [(0, 1), (1, 0), (0, 2), (2, 0), (1, 2), (2, 1), (0, 1)], "half", feat)


def test_more_items_than_the_list_ends_at():
    """70,032 passes, nearly all of them spread: a list of 65,536 items, the other passes whole."""
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(7)
    x = rng.uniform(0.0, 40.0, size=(31120, 3))
    pts = [(x[:n] + rng.uniform(-0.1, 0.1, size=(n, 3))).astype(np.float32) for n in (31120, 4000)]
    feats = [rng.uniform(0.1, 1.0, size=(len(p), 4)).astype(np.float32) for p in pts]
    poses = np.stack([ident(), ident()])
    with rkhsba.Context(ell=0.1, cell_subdiv=3, pass_points=16) as ctx:
        ctx.build_neighbors(pts, feats, "dense")
        _, one, n_one = ctx.eval_loss_noalloc(poses, [(0, 1)])
        for E in (1, 36):
            _, Fe, n = ctx.eval_loss(poses, [(0, 1)] * E)
            assert n == E * n_one and n > 0
            np.testing.assert_array_equal(Fe, np.repeat(one, E))

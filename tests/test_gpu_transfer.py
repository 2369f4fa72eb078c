"""Results and inputs that travel as one small transfer or as copies, on both sides of the limits: 3,584 bytes of
poses in one launch (37 frames) and 14,336 in four (149), 16,384 bytes of per-edge losses (1,024 edges) or of histories.
The values are the same calls' on few frames or edges, bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]


def scene(K, n=20):
    rng = np.random.default_rng(K)
    pts = [rng.uniform(0.0, 0.3, size=(n, 3)).astype(np.float32) for _ in range(K)]
    feats = [rng.integers(0, 3, size=n).astype(np.uint16) for _ in range(K)]
    return pts, feats, np.stack([oracle.se3_exp(rng.normal(scale=0.02, size=6)) for _ in range(K)])


@pytest.mark.parametrize("K", [2, 36, 37, 38, 74, 149, 150, 200])
def test_poses_of_many_frames(K):
    from paper_2403_01254_amd import rkhsba
    pts, feats, poses = scene(K)
    with rkhsba.Context(ell=0.15) as ctx:
        ctx.build_neighbors(pts, feats)
        edges = [(K - 1, K - 2), (0, 1), (K - 2, K - 1)]
        total, per_edge, pairs = ctx.eval_loss(poses, edges)
        got, loss, counts = ctx.gn_step(poses, edges, 0)
        np.testing.assert_array_equal(got, poses)  # 0 iterations: the poses come back as they went
        assert counts[0] == pairs and loss[0] == pytest.approx(total, rel=1e-14)
    few = [0, 1, K - 2, K - 1] if K > 2 else [0, 1]
    with rkhsba.Context(ell=0.15) as ctx:
        ctx.build_neighbors([pts[k] for k in few], [feats[k] for k in few])
        last = len(few) - 1
        want = ctx.eval_loss(poses[few], [(last, last - 1), (0, 1), (last - 1, last)])
    np.testing.assert_array_equal(per_edge, want[1])
    assert pairs == want[2]


@pytest.mark.parametrize("E", [1, 64, 65, 1023, 1024, 1025, 2500])
def test_losses_of_many_edges(E):
    from paper_2403_01254_amd import rkhsba
    pts, feats, poses = scene(5)
    pool = [(m, n) for m in range(5) for n in range(5) if m != n]
    with rkhsba.Context(ell=0.15) as ctx:
        ctx.build_neighbors(pts, feats)
        single = {e: ctx.eval_loss(poses, [e]) for e in pool}
        edges = [pool[(7 * k) % len(pool)] for k in range(E)]
        total, per_edge, pairs = ctx.eval_loss(poses, edges)
    np.testing.assert_array_equal(per_edge, [single[e][1][0] for e in edges])
    assert pairs == sum(single[e][2] for e in edges)
    assert total == pytest.approx(sum(per_edge), rel=1e-12)


@pytest.mark.parametrize("n_iter", [1, 900, 1100])
def test_long_histories(n_iter):
    from paper_2403_01254_amd import rkhsba
    pts, feats, poses = scene(2)
    with rkhsba.Context(ell=0.15, damping_rel=1e-3) as ctx:
        ctx.build_neighbors(pts, feats)
        got, loss, pairs = ctx.gn_step(poses, [(0, 1)], n_iter)
        _, short, short_pairs = ctx.gn_step(poses, [(0, 1)], 1)
        assert len(loss) == n_iter + 1
        np.testing.assert_array_equal(loss[:1], short[:1])
        np.testing.assert_array_equal(pairs[:2], short_pairs)
        final, _, n = ctx.eval_loss(got, [(0, 1)])
        assert loss[-1] == pytest.approx(final, rel=1e-6)

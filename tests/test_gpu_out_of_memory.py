"""A call whose scratch does not fit the card fails with RKHSBA_ENOMEM, and the calls after it give what they gave
before, also on edge lists that were laid out before the failure (its scratch buffers are gone then)."""
import numpy as np
import pytest
import torch

from helpers import ident

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]


def test_calls_after_a_failed_one():
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(0)
    n = 3_000_000
    x = rng.uniform(0.0, 100.0, size=(n, 3)).astype(np.float32)
    pts = [x, (x + rng.normal(scale=0.05, size=x.shape)).astype(np.float32)]
    feats = [rng.uniform(0.1, 1.0, size=(n, 3)).astype(np.float32) for _ in range(2)]
    poses = np.stack([ident(), ident()])
    free, total = torch.cuda.mem_get_info()
    # ten moments of four bytes an entry: more than the whole card, in an edge list below the limit on entries
    E = int(1.02 * total / 40 / n)
    assert 4 * (2**31 - 1) > E * n and free > total // 2
    with rkhsba.Context(ell=0.1, cell_subdiv=1, pass_points=16, damping_rel=1e-3) as ctx:
        ctx.build_neighbors(pts, feats, "dense")
        want = ctx.eval_loss(poses, [(0, 1)]), ctx.gn_step(poses, [(0, 1)], 2)
        assert want[0][2] > n // 2
        with pytest.raises(rkhsba.RkhsbaError) as err:
            ctx.eval_loss(poses, [(0, 1)] * E)
        assert err.value.code == rkhsba.ENOMEM
        for _ in range(2):
            got = ctx.eval_loss(poses, [(0, 1)]), ctx.gn_step(poses, [(0, 1)], 2)
            for a, b in zip(got[0] + got[1], want[0] + want[1]):
                np.testing.assert_array_equal(a, b)

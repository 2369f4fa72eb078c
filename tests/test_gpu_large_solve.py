"""Gauss-Newton steps of graphs of more than 128 unknowns by each route: the block-sparse elimination, the dense one that
it hands nearly free directions to, and the dense one for graphs without a plan (solve_plan.h, asked on the host): panels
too tall for LDS (more than 513 unknowns), and smaller systems with whole 32-row chunks of zeros."""
import os
import subprocess

import numpy as np
import pytest

import oracle
from helpers import ROOT

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]

MAIN = r"""
#include "solve_plan.h"
#include <cstdio>
int main() {
  int n, E;
  if (std::scanf("%d %d", &n, &E) != 2) return 1;
  std::vector<uint8_t> adj((size_t)n * n, 0);
  for (int k = 0, a, b; k < E; ++k) {
    if (std::scanf("%d %d", &a, &b) != 2) return 1;
    if (a >= 0 && b >= 0) adj[(size_t)a * n + b] = adj[(size_t)b * n + a] = 1;
  }
  std::printf("%zu\n", n > rkhsba::kSparseMaxFrames ? (size_t)0 : rkhsba::sparse_plan(n, adj).size());
}
"""


@pytest.fixture(scope="module")
def has_plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2403_01254_amd", "csrc"),
                    str(d / "main.cpp"), "-o", str(d / "main")], check=True)

    def ask(K, edges):  # frame 0 fixed
        text = f"{K - 1} {len(edges)}\n" + "\n".join(f"{m - 1} {n - 1}" for m, n in edges)
        return int(subprocess.run([str(d / "main")], input=text, check=True, capture_output=True, text=True).stdout) > 0

    return ask


def clouds(rng, K, n, offset=0.0, size=0.4):
    pts = [rng.uniform(0.0, size, size=(n, 3)) + [offset * k, 0.0, 0.0] for k in range(K)]
    return [p.astype(np.float32) for p in pts], [rng.uniform(0.1, 1.0, size=(n, 3)).astype(np.float32) for _ in range(K)]


def near(K, reach):
    return [(k, k + d) for k in range(K) for d in range(1, reach + 1) if k + d < K]


def cliques(K):
    """Two complete graphs, joined by one edge."""
    h = K // 2
    return ([(m, n) for m in range(h) for n in range(m + 1, h)] + [(h - 1, h)] +
            [(m, n) for m in range(h, K) for n in range(m + 1, K)])


@pytest.mark.parametrize("K,graph", [(200, "near"), (88, "all"), (80, "cliques"), (86, "cliques"), (24, "cliques")])
def test_dense_step(K, graph, has_plan):
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(K)
    edges = near(K, 3) if graph == "near" else cliques(K) if graph == "cliques" else near(K, K)
    assert has_plan(K, edges) == (K == 24)
    pts, feats = clouds(rng, K, 12)
    poses = np.stack([oracle.se3_exp(rng.normal(scale=0.02, size=6)) for _ in range(K)])
    damping = 1e-2
    with rkhsba.Context(ell=0.15, damping_rel=damping) as ctx:
        ctx.build_neighbors(pts, feats, "dense")
        H, b, _, _ = ctx.accumulate_normal_eqs(poses, edges)
        got, _, _ = ctx.gn_step(poses, edges, 1)
    H, b = H[6:, 6:], b[6:]
    n = len(b)
    delta = np.linalg.solve(H + damping * np.trace(H) / n * np.eye(n), -b)
    # the condition number is at most n / damping + 1, the elimination's relative error some n eps times that
    tol = 4.0 * n * n / damping * np.finfo(float).eps * np.linalg.norm(delta) + 1e-14
    for k in range(1, K):
        R, t, step = poses[k, :9].reshape(3, 3), poses[k, 9:], oracle.se3_exp(delta[6 * k - 6:6 * k])
        np.testing.assert_allclose(got[k, :9].reshape(3, 3), R @ step[:9].reshape(3, 3), rtol=0.0, atol=tol)
        np.testing.assert_allclose(got[k, 9:], R @ step[9:] + t, rtol=0.0, atol=tol)


@pytest.mark.parametrize("line", [True, False])
@pytest.mark.parametrize("K", [32, 48])
def test_nearly_free_directions_go_to_the_dense_elimination(K, line, has_plan):
    """A chain, and the same chain with edges between frames too far apart for a pair: they add exact zeros to the same
    H and b, and take the plan away.  Clouds along one line leave the rotation about it nearly free; there both
    eliminations are the dense one, and poses and pair counts the same bits.  Well-posed chains keep their plan, and
    their poses agree to rounding."""
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(K)
    chain = near(K, 2)
    far = [(m, n) for m in range(K) for n in range(m + 5, K)]
    assert has_plan(K, chain) and not has_plan(K, chain + far)
    pts = []
    for k in range(K):
        s = rng.uniform(0.5 * k, 0.5 * k + 1.2, size=40)
        if line:
            pts.append(np.outer(s, [0.48, 0.6, 0.64]) + rng.normal(scale=3e-5, size=(40, 3)))
        else:
            pts.append(np.c_[s, rng.uniform(0.0, 0.4, size=(40, 2))])
    pts = [p.astype(np.float32) for p in pts]
    feats = [rng.uniform(0.1, 1.0, size=(40, 3)).astype(np.float32) for _ in range(K)]
    poses = np.stack([oracle.se3_exp(np.r_[rng.normal(scale=0.01, size=3), np.zeros(3)]) for _ in range(K)])
    with rkhsba.Context(ell=0.15) as ctx:
        ctx.build_neighbors(pts, feats, "dense")
        Hc, bc, Fc, nc = ctx.accumulate_normal_eqs(poses, chain)
        Hf, bf, Ff, nf = ctx.accumulate_normal_eqs(poses, chain + far)
        np.testing.assert_array_equal(Hc, Hf)
        np.testing.assert_array_equal(bc, bf)
        assert nc == nf > 0
        a = ctx.gn_step(poses, chain, 3)
        b = ctx.gn_step(poses, chain + far, 3)
    if line:
        np.testing.assert_array_equal(a[0], b[0])
    else:
        np.testing.assert_allclose(a[0], b[0], rtol=0.0, atol=1e-10)
    np.testing.assert_array_equal(a[2], b[2])


def test_plan_follows_the_edge_list(has_plan):
    """One set of frames stepped with several edge lists in turn, with and without a plan: each as in a fresh context."""
    from paper_2403_01254_amd import rkhsba
    K = 40
    rng = np.random.default_rng(0)
    pts, feats = clouds(rng, K, 20)
    poses = np.stack([oracle.se3_exp(rng.normal(scale=0.02, size=6)) for _ in range(K)])
    lists = [near(K, 1), near(K, 3), near(K, K), near(K, 3)[::-1], [(n, m) for m, n in near(K, 1)]]
    assert [has_plan(K, e) for e in lists] == [True, True, False, True, True]

    def context():
        ctx = rkhsba.Context(ell=0.15, damping_rel=1e-3)
        ctx.build_neighbors(pts, feats, "dense")
        return ctx

    want = []
    for e in lists:
        with context() as ctx:
            want.append(ctx.gn_step(poses, e, 2))
    with context() as ctx:
        for k in (0, 1, 2, 1, 3, 4, 0, 2, 4, 0):
            for x, y in zip(ctx.gn_step(poses, lists[k], 2), want[k]):
                np.testing.assert_array_equal(x, y)

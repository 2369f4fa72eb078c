"""The rounding of a Gauss-Newton step: H's blocks of one edge, and the solve, against their documented order of fused
multiply-adds on the CPU.  Clouds along a line leave the rotation about it nearly free (a reduced H with eigenvalues
around mu): another order of the same solve moves the poses by 1e-9 and more there, and later pair counts with them,
while the documented one is met to the rounding of the pose update."""
import math

import numpy as np
import pytest

import oracle

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]

DAMPING = 1e-10  # the default


def fma(a, b, c):
    """round(a b + c), exactly: integers on a common power of two."""
    if a == 0.0 or b == 0.0:
        return c
    (ma, ea), (mb, eb), (mc, ec) = math.frexp(a), math.frexp(b), math.frexp(c)
    p, ep = int(math.ldexp(ma, 53)) * int(math.ldexp(mb, 53)), ea + eb - 106
    q, eq = int(math.ldexp(mc, 53)), ec - 53
    e = min(ep, eq)
    return math.ldexp(float((p << (ep - e)) + (q << (eq - e))), e)


def solve_by_columns(H, b, mu):
    """(H + mu I) x = -b without square roots, column by column: the later row divided by the pivot, the earlier one
    not, -b as the last row."""
    n = len(b)
    A = [[float(H[i, k]) for k in range(i + 1)] for i in range(n)] + [[-float(v) for v in b]]
    for i in range(n):
        A[i][i] += mu
    for j in range(n):
        inv = 1.0 / A[j][j]
        scaled = [row[j] * inv for row in A[j + 1:]]
        for i in range(j + 1, n + 1):
            for k in range(j + 1, min(i, n - 1) + 1):
                A[i][k] = fma(-scaled[i - j - 1], A[k][j], A[i][k])
        for i in range(j + 1, n + 1):
            A[i][j] = scaled[i - j - 1]
    x = A[n]
    for j in range(n - 1, 0, -1):
        for t in range(j):
            x[t] = fma(-A[j][t], x[j], x[t])
    return np.array(x)


def line_clouds(rng, K, n=60):
    """Points within some 3e-5 of a line in a general position."""
    s = np.sort(rng.uniform(-1.0, 1.0, size=n))
    pts = []
    for _ in range(K):
        p = np.outer(s + rng.normal(scale=0.01, size=n), [0.48, 0.6, 0.64]) + [2.0, -1.0, 3.0]
        pts.append((p + rng.normal(scale=3e-5, size=(n, 3))).astype(np.float32))
    feats = [rng.uniform(0.1, 1.0, size=(n, 3)).astype(np.float32) for _ in range(K)]
    return pts, feats


def spread_clouds(rng, K, n=60):
    pts = [rng.uniform(-0.3, 0.3, size=(n, 3)).astype(np.float32) for _ in range(K)]
    feats = [rng.uniform(0.1, 1.0, size=(n, 3)).astype(np.float32) for _ in range(K)]
    return pts, feats


@pytest.mark.parametrize("edges", ["ring", "many"])  # one workgroup takes the whole step, or the solve alone (65 edges)
@pytest.mark.parametrize("clouds", [line_clouds, spread_clouds])
@pytest.mark.parametrize("K", [2, 3, 8, 22])
def test_solve_order(K, clouds, edges):
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(K)
    pts, feats = clouds(rng, K)
    poses = np.stack([oracle.se3_exp(np.r_[rng.normal(scale=0.02, size=3), np.zeros(3)]) for _ in range(K)])
    e = [(k, (k + 1) % K) for k in range(K)] if K > 2 else [(0, 1)]
    if edges == "many":
        e = (e * 65)[:65]
    with rkhsba.Context(ell=0.1, damping_rel=DAMPING) as ctx:
        ctx.build_neighbors(pts, feats, "dense")
        H, b, _, _ = ctx.accumulate_normal_eqs(poses, e)
        got, _, _ = ctx.gn_step(poses, e, 1)
    H, b = H[6:, 6:], b[6:]
    n = len(b)
    # the trace as a wavefront sums it: lanes 32, 16, .. 1 apart, the two halves of more than 64 entries after another
    tr = 0.0
    for h in range(0, n, 64):
        v = np.zeros(64)
        v[:min(64, n - h)] = np.diag(H)[h:h + 64]
        for o in (32, 16, 8, 4, 2, 1):
            v = v + v[np.arange(64) ^ o]
        tr += v[0]
    delta = solve_by_columns(H, b, DAMPING * tr / n)
    size = np.abs(delta).max()
    if clouds is line_clouds:  # the scene does tell one order from another
        flipped = solve_by_columns(H[::-1, ::-1], b[::-1], DAMPING * tr / n)[::-1]
        assert np.abs(flipped - delta).max() > 1e-9
    for k in range(1, K):
        R, t = poses[k, :9].reshape(3, 3), poses[k, 9:]
        step = oracle.se3_exp(delta[6 * k - 6:6 * k])
        # some 30 operations on numbers up to 1 + |delta|, each rounded once
        tol = 32 * np.finfo(float).eps * (1.0 + size)
        np.testing.assert_allclose(got[k, :9].reshape(3, 3), R @ step[:9].reshape(3, 3), rtol=0.0, atol=tol)
        np.testing.assert_allclose(got[k, 9:], R @ step[9:] + t, rtol=0.0, atol=tol)


def relative_rotation(Tm, Tn):
    return [[fma(Tn[6 + a], Tm[6 + c], fma(Tn[3 + a], Tm[3 + c], Tn[a] * Tm[c])) for c in range(3)] for a in range(3)]


@pytest.mark.parametrize("seed", range(6))
def test_edge_blocks(seed):
    """One edge: b_m = R_mn B, and H_mn's R_mn [S] and -[A x] R_mn, from the B, S and A x that b_n, H_nn and H_mm hold."""
    from paper_2403_01254_amd import rkhsba
    rng = np.random.default_rng(seed)
    turn = oracle.se3_exp(np.r_[np.zeros(3), rng.normal(size=3)])[:9].reshape(3, 3)
    pts = [rng.uniform(-0.5, 0.5, size=(400, 3)).astype(np.float32) for _ in range(2)]
    pts[1] = (pts[1].astype(np.float64) @ turn).astype(np.float32)
    feats = [rng.uniform(0.1, 1.0, size=(400, 3)).astype(np.float32) for _ in range(2)]
    first = oracle.se3_exp(rng.normal(size=6))
    step = oracle.se3_exp(rng.normal(scale=0.05, size=6))
    R0 = first[:9].reshape(3, 3)
    poses = np.stack([first, np.r_[(R0 @ step[:9].reshape(3, 3) @ turn).reshape(9), R0 @ step[9:] + first[9:]]])
    with rkhsba.Context(ell=0.1) as ctx:
        ctx.build_neighbors(pts, feats, "dense")
        H, b, _, _ = ctx.accumulate_normal_eqs(poses, [(0, 1)])
    Rnm = relative_rotation(poses[0].tolist(), poses[1].tolist())
    R = [[Rnm[c][r] for c in range(3)] for r in range(3)]
    Ax, S, B = -H[0:3, 3:6], -H[6:9, 9:12], -b[6:9]  # (cross-product matrices)

    def row_dot(r, v):
        return fma(R[r][2], float(v[2]), fma(R[r][0], float(v[0]), R[r][1] * float(v[1])))

    for r in range(3):
        assert b[r] == row_dot(r, B)
        for c in range(3):
            assert H[r, 9 + c] == row_dot(r, S[:, c]), (r, c)
            v = 0.0
            for a in range(3):
                v = fma(float(Ax[r, a]), R[a][c], v)
            assert H[3 + r, 6 + c] == -v, (r, c)

"""GPU kernels at the sizes where their tiling and dispatch change, against the oracle."""
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_1307_2666_amd as hif
from oracle.idqr import interp_decomp
from oracle.kernels import Operator
from workloads import grid_points

from test_gpu_parity import _check_id

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(40, 31), (256, 32), (257, 33), (511, 96), (4096, 64), (4097, 65), (4353, 129),
                                 (8200, 95), (32768, 48)])
def test_row_compression_tree_edges(m, n):
    # Row compression of problems at the edges of its tree: one chunk of at
    # most 256 rows, one group of at most 16 chunks, several groups; last
    # panels of fewer than 32 columns; three unequal problems in one batch.
    # The column scales make the pivots unique, so that the ID of R0 has the
    # oracle's skeleton and T.
    rng = np.random.default_rng(m + n)
    cases = []
    for mm, nn in ((m, n), (max(n + 1, m - 37), n), (m // 2 + n, max(2, n - 5))):
        cases.append(rng.standard_normal((mm, nn)) * (10.0 ** (-9.0 * np.arange(nn) / nn))[rng.permutation(nn)])
    tol = 1e-6
    out = hif.id_batched([torch.tensor(Y) for Y in cases], [tol] * len(cases))
    for Y, (sk, rd, T) in zip(cases, out):
        osk, _, oT = interp_decomp(Y, tol)
        _check_id(Y, tol, True, sk.numpy(), rd.numpy(), T.numpy(), osk, oT)


@pytest.mark.parametrize("m,n", [(128, 40), (129, 40),                      # a chunk by 2 waves, by 4
                                 (1024, 40), (1025, 40), (2048, 40), (2049, 40),  # stacks of 4, 5, 8 and 9 chunk factors
                                 (16384, 33), (16385, 33)])                    # roots of 4 and 5 groups
def test_row_compression_node_waves(m, n):
    # The waves of a tree node follow from the tallest problem of a batch; one
    # of nearly its height and one of a third share it here.
    rng = np.random.default_rng(m + n)
    cases = []
    for mm in (m, m - 1, m // 3 + n):
        cases.append(rng.standard_normal((mm, n)) * (10.0 ** (-9.0 * np.arange(n) / n))[rng.permutation(n)])
    tol = 1e-6
    out = hif.id_batched([torch.tensor(Y) for Y in cases], [tol] * len(cases))
    for Y, (sk, rd, T) in zip(cases, out):
        osk, _, oT = interp_decomp(Y, tol)
        _check_id(Y, tol, True, sk.numpy(), rd.numpy(), T.numpy(), osk, oT)


@pytest.mark.parametrize("sizes", [
    [(64, 64), (65, 65), (16, 16), (17, 3), (1, 1)],       # one panel, a column past it
    [(130, 64), (130, 65), (128, 63), (200, 129)],         # panels that end at, past and short of 64 columns
    [(513, 100), (1025, 80), (300, 300)],                  # every thread count of the register panel
    [(2049, 70), (500, 200)],                              # a panel over the registers beside one within them
])
def test_lu_batched_panel_edges(sizes):
    # P A = L U over the first r columns to the backward error bound of the
    # elimination, |P A - L U| <= n u |L| |U| (tripled: the multipliers are
    # products with the pivot's rounded reciprocal), entry by entry, and the
    # pivots of partial pivoting: |L| <= 1 (up to the rounding of the
    # multipliers) among the candidate rows.
    rng = np.random.default_rng(sum(n + r for n, r in sizes))
    mats = [rng.standard_normal((n, n)) for n, _ in sizes]
    out, pv, zero = hif.lu_batched([torch.tensor(M) for M in mats], [r for _, r in sizes])
    assert not zero
    u = np.finfo(float).eps / 2
    for M, (n, r), F, piv in zip(mats, sizes, out, pv):
        F, piv = F.numpy(), piv.numpy()
        P = M.copy()
        for j, p in enumerate(piv):
            assert j <= p < r
            P[[j, p]] = P[[p, j]]
        L = np.tril(F[:, :r], -1) + np.eye(n, r)
        U = np.triu(F[:r])
        R = L @ U
        R[r:, r:] += F[r:, r:]
        bound = np.abs(L) @ np.abs(U)
        bound[r:, r:] += np.abs(F[r:, r:])
        # the comparison's own product is as inexact again
        assert np.all(np.abs(P - R) <= 4 * (r + 2) * u * bound)
        assert np.abs(L[:r]).max() <= 1 + 2 * u


@pytest.mark.parametrize("sizes", [
    [(64, 64), (20, 5)], [(30, 30), (30, 10)], [(16, 16), (17, 3), (17, 17)],  # all columns of one, few of another
    [(40, 1), (64, 64), (64, 63)], [(2, 1), (2, 2)],
])
def test_lu_batched_small_blocks_of_unequal_depth(sizes):
    # blocks of one panel: the interchanges and U12 of a block eliminated in
    # part, beside one eliminated whole
    test_lu_batched_panel_edges(sizes)


def test_lu_batched_singular_panel_reports_and_stays_in_bounds():
    # a zero column inside the second panel: the status is set, and the
    # panels after it find only interchanges within the block
    M = np.random.default_rng(5).standard_normal((200, 200))
    M[:, 90] = 0.0
    _, _, zero = hif.lu_batched([torch.tensor(M)], [200])
    assert zero


@pytest.mark.parametrize("n,col,value", [(2100, 0, 0.0), (2305, 0, np.nan), (2100, 17, 0.0), (2100, 18, 0.0)])
def test_lu_batched_tall_singular_panel_reports_and_stays_in_bounds(n, col, value):
    # a column without a pivot in a panel over many workgroups, the first
    # column of all among them (nothing is left of an earlier step then): the
    # status is set, every interchange is one within the block, and the block
    # beside it is factored as beside a nonsingular one
    rng = np.random.default_rng(n + col)
    whole, good = rng.standard_normal((n, n)), rng.standard_normal((2200, 2200))
    bad = whole.copy()
    bad[:, col] = value
    out, pv, zero = hif.lu_batched([torch.tensor(bad), torch.tensor(good)], [600, 600])
    assert zero
    assert np.all((pv[0].numpy() >= 0) & (pv[0].numpy() < 600))
    ref, pvr, zero = hif.lu_batched([torch.tensor(whole), torch.tensor(good)], [600, 600])
    assert not zero
    assert torch.equal(out[1], ref[1]) and torch.equal(pv[1], pvr[1])


@pytest.mark.parametrize("m,n,decay,tol", [
    (128, 128, 5.0, 1e-3), (140, 129, 12.0, 1e-9),   # one and two chunks; several Gram matrices
    (300, 1024, 9.0, 1e-6), (300, 1025, 9.0, 1e-6),  # the last width with the Cholesky rows in registers
    (200, 2049, 6.0, 1e-4), (200, 4096, 6.0, 1e-4),  # several columns per thread
    (1, 200, 3.0, 1e-2), (33, 400, 3.0, 1e-8),       # fewer rows than a block; a block of one column after a full one
])
def test_blocked_pivoted_qr_edges(m, n, decay, tol):
    # The pivots come from Gram matrices good to about 1e-10 of the largest
    # squared norm; random columns of separated scales are further apart, so
    # the skeleton and T are the oracle's.  Two problems share the batch.
    rng = np.random.default_rng(m * 7 + n)
    cases = []
    for mm, nn in ((m, n), (max(1, m - 1), max(128, n - 3))):
        cases.append(rng.standard_normal((mm, nn)) * (10.0 ** (-decay * np.arange(nn) / nn))[rng.permutation(nn)])
    out = hif.id_batched([torch.tensor(Y) for Y in cases], [tol] * len(cases))
    for Y, (sk, rd, T) in zip(cases, out):
        osk, _, oT = interp_decomp(Y, tol)
        _check_id(Y, tol, True, sk.numpy(), rd.numpy(), T.numpy(), osk, oT)


@pytest.mark.parametrize("m,n", [(200, 150), (64, 1100), (300, 4096)])
@pytest.mark.parametrize("rank", [1, 31, 32, 33, 63])
def test_blocked_pivoted_qr_of_low_rank(m, n, rank):
    # Rank at, before and after the ends of blocks, the rest eight digits below
    # the tolerance or zero: what is left then stops the choice.  The rank is the
    # oracle's and T within its bounds.  Unequal ranks share the batch.
    rng = np.random.default_rng(m + n + rank)
    cases = []
    for nn, r, noise in ((n, rank, 0.0), (max(128, n - 7), max(1, rank - 2), 1e-14), (n, min(rank + 40, 63), 1e-14)):
        U = np.linalg.qr(rng.standard_normal((m, r)))[0]
        Y = (U * 10.0 ** (-3.0 * np.arange(r) / r)) @ rng.standard_normal((r, nn))
        cases.append(Y + noise * rng.standard_normal((m, nn)))
    out = hif.id_batched([torch.tensor(Y) for Y in cases], [1e-6] * len(cases))
    for Y, (sk, rd, T) in zip(cases, out):
        osk, _, oT = interp_decomp(Y, 1e-6)
        assert sk.numel() == len(osk)
        _check_id(Y, 1e-6, False, sk.numpy(), rd.numpy(), T.numpy(), osk, oT)


@pytest.mark.parametrize("m,n", [(600, 40), (600, 150), (600, 600), (4400, 300)])
def test_reflectors_of_columns_whose_squares_underflow(m, n):
    # In the first panel's chunks of rows: the second holds three rows of rank 1,
    # so that after one column only rounding errors of rounding errors are left,
    # the last four rows down to where squares underflow, and one column is as
    # small altogether.  All of it is below the tolerance beside the other rows:
    # skeleton and T are the oracle's.
    rng = np.random.default_rng(m + n)
    nck = (m + 255) // 256
    cases = []
    for _ in range(2):
        Y = rng.standard_normal((m, n)) * (10.0 ** (-9.0 * np.arange(n) / n))[rng.permutation(n)]
        lo, hi, last = m // nck, 2 * m // nck, (nck - 1) * m // nck
        Y[lo:hi] = 0.0
        Y[lo + 50:lo + 53] = 1e-30 * rng.standard_normal((3, 1)) * rng.standard_normal(n)
        Y[last:] = 0.0
        Y[last + 40:last + 44] = np.array([1e-40, 1e-90, 1e-145, 1e-157])[:, None] * rng.standard_normal((4, n))
        Y[:, n // 3] = 1e-158 * rng.standard_normal(m)
        cases.append(Y)
    out = hif.id_batched([torch.tensor(Y) for Y in cases], [1e-6] * len(cases))
    for Y, (sk, rd, T) in zip(cases, out):
        osk, _, oT = interp_decomp(Y, 1e-6)
        _check_id(Y, 1e-6, True, sk.numpy(), rd.numpy(), T.numpy(), osk, oT)


def test_blocked_pivoted_qr_zero_tied_and_nonfinite_columns():
    # Zero columns are never pivots; of equal columns the lowest is chosen
    # first and the others vanish; a column of NaN is never chosen and does not
    # stop the others.
    rng = np.random.default_rng(4)
    Y = np.repeat(rng.standard_normal((150, 40)) * 10.0 ** (-np.arange(40) / 10.0), 5, axis=1)
    Y[:, 17] = 0.0
    (sk, rd, T), = hif.id_batched([torch.tensor(Y)], [1e-9])
    osk, _, oT = interp_decomp(Y, 1e-9)
    assert sk.numel() == 40 and set((sk.numpy() // 5).tolist()) == set(range(40))
    assert np.all(sk.numpy() % 5 <= 1) and 17 not in sk.tolist()
    assert np.linalg.norm(Y[:, rd.numpy()] - Y[:, sk.numpy()] @ T.numpy()) <= 1e-9 * np.linalg.norm(Y)
    Y[:, 3] = np.nan
    (sk, rd, T), = hif.id_batched([torch.tensor(Y)], [1e-9])
    assert sk.numel() == 40 and 3 not in sk.tolist()


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("n,nrhs", [(1, 1), (63, 2), (65, 3), (257, 9), (1000, 6), (32767, 4), (32768, 5),
                                    (262143, 1), (262144, 7)])
def test_matvec_sizes_and_right_hand_sides(d, n, nrhs):
    # The product at the sizes where its split of targets and sources changes
    # and for every number of right-hand sides a pass takes, against sampled
    # rows: a row's sum of n terms is off by at most n u of the sum of their
    # magnitudes, each term by 8 u (the kernel within 2 ulp, the distance and
    # weights); G is small near r = 1, so its own scale is kept above 1e-3.
    gen = np.random.default_rng(n + 10 * nrhs + d)
    pts = gen.random((n, d))
    w, s, a, b, c = (0.5 + gen.random(n) for _ in range(5))
    x = gen.standard_normal((nrhs, n))
    t = lambda v: torch.tensor(v, device="cuda:0")  # noqa: E731
    y = hif.matvec(t(pts), t(x), a=t(a), b=t(b), c=t(c), weights=t(w), selfk=t(s)).cpu().numpy()
    u = np.finfo(float).eps / 2
    for i in sorted({0, n - 1, n // 2, *gen.integers(0, n, 6).tolist()}):
        r = np.sqrt(((pts[i] - pts) ** 2).sum(1))
        r[i] = 1.0
        G = -np.log(r) / (2 * np.pi) if d == 2 else 1.0 / (4 * np.pi * r)
        G[i] = 0.0
        K = G * w
        K[i] = s[i]
        ref = a[i] * x[:, i] + b[i] * ((K * c) * x).sum(1)
        mag = np.abs(a[i] * x[:, i]) + b[i] * ((np.maximum(np.abs(K), 1e-3 * w) * c) * np.abs(x)).sum(1)
        assert np.all(np.abs(y[:, i] - ref) <= (2 * n * u + 16 * u) * mag)


@pytest.mark.parametrize("n", [3, 64, 65, 40000])  # one, both and neither of the splits' last tiles full
@pytest.mark.parametrize("d", [2, 3])
def test_matvec_points_outside_the_unit_box(d, n):
    # The product checks no coordinates: points anywhere give the formula's
    # sum, at (2, 3) and (2, 3, 4) as elsewhere, and in 3D a pair whose squared
    # distance overflows counts as infinitely far.  Tolerance of
    # test_matvec_sizes_and_right_hand_sides, all weights one.
    gen = np.random.default_rng(n + d)
    pts = gen.random((n, d))
    pts[0] = 2.0 + np.arange(d)
    if d == 3:
        pts[1] = (1e200, 0.5, 0.5)
    x = gen.standard_normal((2, n))
    t = lambda v: torch.tensor(v, device="cuda:0")  # noqa: E731
    y = hif.matvec(t(pts), t(x), weights=t(np.ones(n)), selfk=t(np.ones(n))).cpu().numpy()
    u = np.finfo(float).eps / 2
    for i in {0, 1, 2, n - 1}:
        with np.errstate(over="ignore"):
            r = np.sqrt(((pts[i] - pts) ** 2).sum(1))
        r[i] = 1.0
        K = -np.log(r) / (2 * np.pi) if d == 2 else 1.0 / (4 * np.pi * r)
        K[i] = 1.0
        assert np.all(np.abs(y[:, i] - (K * x).sum(1)) <= (2 * n * u + 16 * u) * (np.maximum(np.abs(K), 1e-3) * np.abs(x)).sum(1))


@pytest.mark.parametrize("n,d,leaf,eps", [(16, 2, 64, 1e-9), (28, 2, 64, 1e-9), (40, 2, 16, 1e-9), (64, 2, 64, 1e-10),
                                          (12, 3, 64, 1e-6), (20, 3, 64, 1e-6)])
def test_sweeps_top_sizes_and_right_hand_sides(n, d, leaf, eps):
    # The four sweeps of a non-symmetric operator over top blocks from below
    # one 64-row block of the chained solve to many, and over records of few
    # large groups.  F^-1 F x = x and <F^T x, y> = <x, F y> to rounding times
    # the size of the operator's inverse (about 1 here: a well conditioned
    # second-kind operator), and right-hand sides taken together, in passes of
    # 1, 4 and 8, give each one's own result.
    rng = np.random.default_rng(n * d)
    g = (np.arange(n) + 0.5) / n
    pts = np.stack(np.meshgrid(*[g] * d, indexing="ij"), -1).reshape(-1, d)
    N = n ** d
    t = lambda v: torch.tensor(v, device="cuda:0")  # noqa: E731
    F = hif.factor(t(pts), eps, leaf, a=t(1.0 + rng.random(N)), b=t(0.5 + rng.random(N)), c=t(0.5 + rng.random(N)),
                   h=1.0 / n)
    x, y = t(rng.standard_normal((9, N))), t(rng.standard_normal((9, N)))
    rel = lambda a, b: (torch.linalg.norm(a - b, dim=1) / torch.linalg.norm(b, dim=1)).max().item()  # noqa: E731
    assert rel(F.solve(F.apply(x)), x) <= 1e-10
    assert rel(F.solve_T(F.apply_T(x)), x) <= 1e-10
    for op, tr in ((F.apply, F.apply_T), (F.solve, F.solve_T)):
        Oy = op(y)
        dot = ((tr(x) * y).sum(1) - (x * Oy).sum(1)).abs() / (torch.linalg.norm(x, dim=1) * torch.linalg.norm(Oy, dim=1))
        assert dot.max().item() <= 1e-12
        for f in (op, tr):
            full = f(x)
            for k in (1, 2, 3, 4, 5):
                assert rel(f(x[:k].clone()), full[:k]) <= 1e-13
            z = x.clone()
            f(z, out=z)  # in place
            assert torch.equal(z, full)
    F.free()


@pytest.mark.parametrize("n,leaf", [(16, 64), (20, 100), (24, 144), (32, 256), (40, 400), (46, 529)])
def test_sweeps_of_large_records_in_one_workgroup(n, leaf):
    # Four cells that hold most of the unknowns as redundant ones: records of up
    # to 64, 128, 256 and more rows that are swept by one workgroup each, whose
    # triangular products take only the columns their rows reach.  The checks
    # are those of the other sizes, and the product is F's own: A x to 10 eps.
    test_sweeps_top_sizes_and_right_hand_sides(n, 2, leaf, 1e-9)
    pts = torch.tensor(grid_points(n, 2), device="cuda:0")
    a = torch.ones(n * n, dtype=torch.float64, device="cuda:0")
    c = 1.0 + pts[:, 1]
    F = hif.factor(pts, 1e-9, leaf, a=a, c=c, h=1.0 / n)
    x = torch.tensor(np.random.default_rng(n).standard_normal((3, n * n)), device="cuda:0")
    Ax = hif.matvec(pts, x, a=a, c=c, h=1.0 / n)
    ATx = hif.matvec(pts, x, a=a, b=c, h=1.0 / n)  # K is symmetric on a uniform grid
    assert (torch.linalg.norm(F.apply(x) - Ax) / torch.linalg.norm(Ax)).item() <= 1e-8
    assert (torch.linalg.norm(F.apply_T(x) - ATx) / torch.linalg.norm(ATx)).item() <= 1e-8
    F.free()


@pytest.mark.parametrize("n", [22, 26, 32])  # cells of 121, 169 and 256 columns: rows as they are, padded, and past 1 KiB
def test_padded_blocks_as_assembled(n):
    # A group's block Y with rows padded in memory: the copy handed out has
    # none, its near-field rows hold the kernel to 12 u of |K| + h^2 / 2 pi
    # (each side within 6 u), and what is built on it still inverts.
    pts = grid_points(n, 2)
    op = Operator.uniform(pts, 1.0 / n)
    F = hif.factor(torch.tensor(pts, device="cuda:0"), 1e-9, n * n // 4, a=torch.tensor(op.a, device="cuda:0"),
                   h=1.0 / n, trace_sublevel=0)
    tr = F.trace()
    gs, ns = tr["group_start"], tr["near_start"]
    assert np.all(np.diff(gs) == n * n // 4)
    u, h2pi = 2.0 ** -53, (1.0 / n) ** 2 / (2 * np.pi)
    for g in range(gs.size - 1):
        dofs, near = tr["group_dofs"][gs[g]:gs[g + 1]], tr["near_dofs"][ns[g]:ns[g + 1]]
        Y = tr["Y"][tr["y_off"][g]:tr["y_off"][g] + near.size * dofs.size].reshape(near.size, dofs.size)
        K = op.kernel_block(near, dofs)
        assert np.all(np.abs(Y - K) <= 12 * u * (np.abs(K) + h2pi)), g
    x = torch.tensor(np.random.default_rng(n).standard_normal((2, n * n)), device="cuda:0")
    assert (torch.linalg.norm(F.solve(F.apply(x)) - x) / torch.linalg.norm(x)).item() <= 1e-10
    F.free()


@pytest.mark.parametrize("n,d,leaf", [(32, 2, 16), (96, 2, 64), (12, 3, 64)])  # small records, a chained top, one over half
def test_recorded_solve_keeps_its_scratch(n, d, leaf):
    # A solve recorded with one right-hand side, then a solve of the same
    # handle with eight (more scratch than was recorded), another factorization
    # (which takes what was released) and a second recorded solve: the replays
    # still give the eager solves, and leave the other factorization alone.
    rng = np.random.default_rng(n + d)
    g = (np.arange(n) + 0.5) / n
    pts = torch.tensor(np.stack(np.meshgrid(*[g] * d, indexing="ij"), -1).reshape(-1, d), device="cuda:0")
    N = n ** d
    t = lambda v: torch.tensor(v, device="cuda:0")  # noqa: E731
    one = torch.ones(N, dtype=torch.float64, device="cuda:0")
    F = hif.factor(pts, 1e-6, leaf, a=one, h=1.0 / n)
    f1, f8 = t(rng.standard_normal((1, N))), t(rng.standard_normal((8, N)))
    u1, u8 = torch.empty_like(f1), torch.empty_like(f8)
    g1 = F.solve_graph(f1, u1)
    ref8 = F.solve(f8)
    g8 = F.solve_graph(f8, u8)
    G = hif.factor(pts, 1e-6, leaf, a=2.0 * one, h=1.0 / n)
    other = G.solve(f1)
    for _ in range(3):
        f1.copy_(t(rng.standard_normal((1, N))))
        ref1 = F.solve(f1)
        want = G.solve(f1)
        for gr in (g1, g8):
            gr.launch()
        torch.cuda.synchronize()
        assert torch.equal(u1, ref1) and torch.equal(u8, ref8)
        assert torch.equal(G.solve(f1), want)
    g1.free()
    assert torch.equal(F.solve(f8), ref8)
    g8.free()
    G.free()
    F.free()
    assert torch.isfinite(other).all()


@pytest.mark.parametrize("a,f,u", [
    (3.0, 1.0, 1.0 / 3.0), (2.0, np.inf, np.inf), (-2.0, np.inf, -np.inf), (1e-10, 1e308, np.inf),
    (3e-310, 1e-310, 1e-310 / 3e-310), (-3e-310, 0.0, 0.0), (1.7e308, 1e308, 1e308 / 1.7e308), (3.0, -np.inf, -np.inf),
])
def test_small_solves_divide_as_division_does(a, f, u):
    # One unknown with A = a: the quotient at the ends of the range, where a
    # product with the reciprocal would give NaN, in both solves and for each
    # number of right-hand sides a wave takes.
    t = lambda v: torch.tensor(v, dtype=torch.float64, device="cuda:0")  # noqa: E731
    F = hif.factor(t([[0.5, 0.5]]), 1e-6, 1, a=t([a]), weights=t([0.0]), selfk=t([0.0]))
    for nrhs in (1, 3, 8):
        x = torch.full((nrhs, 1), f, dtype=torch.float64, device="cuda:0")
        for y in (F.solve(x), F.solve_T(x)):
            assert y.cpu().numpy().ravel().tolist() == [u] * nrhs
    F.free()


@pytest.mark.parametrize("n", [8, 11])  # one diagonal block of 64, two
def test_small_solves_beside_a_subnormal_pivot(n):
    # A dense diagonal block (one leaf, no levels, no weights) whose last entry
    # is subnormal: each unknown is its quotient, within the two roundings of a
    # corrected product with the reciprocal.
    N = n * n
    rng = np.random.default_rng(n)
    a = 1.0 + rng.random(N)
    a[-1] = 3e-310
    f = rng.standard_normal((5, N))
    f[:, -1] *= 1e-310
    t = lambda v: torch.tensor(v, device="cuda:0")  # noqa: E731
    zero = t(np.zeros(N))
    F = hif.factor(t(grid_points(n, 2)), 1e-6, N, a=t(a), weights=zero, selfk=zero)
    for y in (F.solve(t(f)), F.solve_T(t(f))):
        assert np.all(np.abs(y.cpu().numpy() - f / a) <= 2 * np.finfo(float).eps * np.abs(f / a))
    F.free()


@pytest.mark.parametrize("n", [12, 20, 25])
def test_dense_factorization_under_a_tight_memory_cap(n):
    # One leaf, no levels: 8 n^2 bytes of the block and a hundred an unknown
    # (points, coefficients, indices) hold the factorization, 72 more the
    # vectors of 8 right-hand sides.  From there up every cap is enough, with
    # whatever the sweeps keep beside the factors, and the four sweeps are those
    # of a factorization without a cap: to the rounding of two orders of
    # summation, at most 4 N u of the operator's condition (below 50).
    N = n * n
    g = (np.arange(n) + 0.5) / n
    pts = torch.tensor(np.stack(np.meshgrid(g, g, indexing="ij"), -1).reshape(-1, 2), device="cuda:0")
    a = torch.ones(N, dtype=torch.float64, device="cuda:0")
    x = torch.tensor(np.random.default_rng(n).standard_normal((9, N)), device="cuda:0")
    kw = dict(a=a, b=1.0 + pts[:, 0], c=2.0 - pts[:, 1], h=1.0 / n)
    F = hif.factor(pts, 1e-6, N, **kw)
    ref = [F.solve(x), F.solve_T(x), F.apply(x), F.apply_T(x)]
    F.free()
    least = 8 * N * N + 172 * N
    for extra in [0, 8, 64, 72 * N, 3 << 15, *range(1 << 16, 1 << 20, 1 << 16)]:
        F = hif.factor(pts, 1e-6, N, max_bytes=least + extra, **kw)
        for _ in range(2):
            for f, r in zip((F.solve, F.solve_T, F.apply, F.apply_T), ref):
                assert (torch.linalg.norm(f(x) - r) / torch.linalg.norm(r)).item() <= 50 * 4 * N * 2.0 ** -53, extra
        u = torch.empty_like(x[:3])
        gr = F.solve_graph(x[:3].clone(), u)
        gr.launch()
        torch.cuda.synchronize()
        assert (torch.linalg.norm(u - ref[0][:3]) / torch.linalg.norm(u)).item() <= 50 * 4 * N * 2.0 ** -53, extra
        gr.free()
        F.free()


def test_group_of_more_columns_than_the_pivot_choice_holds():
    # One leaf of 128 x 129 = 16512 points beside three of 16: its ID has more
    # columns than the pivot choice keeps in registers, and few rows.  A is the
    # identity plus a small integral operator, so apply error and solve
    # residual against the exact product are within 10 eps.
    eps, h = 1e-6, 0.5 / 129
    big = np.stack(np.meshgrid((np.arange(128) + 0.5) * h, (np.arange(129) + 0.5) * h, indexing="ij"), -1).reshape(-1, 2)
    few = np.stack(np.meshgrid(*[(np.arange(4) + 0.5) / 8] * 2, indexing="ij"), -1).reshape(-1, 2)
    pts = np.concatenate([big] + [few + np.array(o) for o in ((0.5, 0.0), (0.0, 0.5), (0.5, 0.5))])
    P = torch.tensor(pts, device="cuda:0")
    a = torch.ones(pts.shape[0], dtype=torch.float64, device="cuda:0")
    F = hif.factor(P, eps, 16512, a=a, h=h)
    st = F.stats()
    assert st["top_size"] < 1000
    x = torch.tensor(np.random.default_rng(6).standard_normal((2, pts.shape[0])), device="cuda:0")
    rel = lambda v, w: (torch.linalg.norm(v - w, dim=1) / torch.linalg.norm(w, dim=1)).max().item()  # noqa: E731
    assert rel(F.apply(x), hif.matvec(P, x, a=a, h=h)) <= 10 * eps
    assert rel(hif.matvec(P, F.solve(x), a=a, h=h), x) <= 10 * eps
    F.free()


_SCARCE = """
import sys
import numpy as np, torch
import paper_1307_2666_amd as hif
rng = np.random.default_rng(2)
cols = lambda n: (10.0 ** (-6.0 * np.arange(n) / n))[rng.permutation(n)]
hif.id_batched([torch.tensor(rng.standard_normal((100, 130)))], [1e-3])  # the library's code on the device
mats = [torch.tensor(rng.standard_normal((500, 4096)) * cols(4096)) for _ in range(int(sys.argv[1]))]
tols = [1e-3] * len(mats)
new = lambda mib: torch.empty(mib << 20, dtype=torch.uint8, device="cuda")
keep = new(2048)  # for the call's own tensors
rest = [new((torch.cuda.mem_get_info()[0] >> 20) - 4096)]
while True:  # what the device really has left
    try:
        rest.append(new(256))
    except torch.OutOfMemoryError:
        break
print("blocks", len(rest), flush=True)
del rest[1:5]
torch.cuda.empty_cache()
del keep
few = hif.id_batched(mats, tols)
del rest
torch.cuda.empty_cache()
many = hif.id_batched(mats, tols)
for x, y in zip(few, many):
    assert all(torch.equal(p, q) for p, q in zip(x, y)) and x[0].numel() > 32
print("equal", len(few))
"""


@pytest.mark.parametrize("count", [8, 9])
def test_blocked_pivoted_qr_where_memory_is_short(count):
    # 1 GiB of device memory left for 8 or 9 Gram matrices of 128 MiB and their
    # problems: they go through in parts, with the results of all together.  A
    # process of its own, whose allocator holds no blocks of earlier calls.
    r = subprocess.run([sys.executable, "-c", _SCARCE, str(count)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and f"equal {count}" in r.stdout, r.stdout + r.stderr

"""The Gram panel at the edges of its 16-column blocks, its row tiles and its
grid (one workgroup, several, many rows per wavefront), and where a sweep ends
inside a block."""

import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
import paper_2608_28941_amd as rrf
from gpu_util import say, to_dev, to_host

pytestmark = pytest.mark.gpu


def _check(Y, tol):
    m, b = Y.shape
    with pytest.MonkeyPatch.context() as mp:
        mp.setenv("RRF_PANEL", "gram")     # (a panel of > 32 columns on its own: the grid)
        p = rrf.Plan(torch.float64, m, b, b)
    with p:
        V, T, tau = (to_host(x) for x in p.panel_qr(to_dev(Y)))
    V_o, tau_o = oracle.geqr2(Y)
    # Householder QR is backward stable: the reflectors agree to cond(Y) u
    # times a modest factor (as the panel tests of the stages state it).
    assert np.max(np.abs(tau - tau_o)) < tol
    assert np.max(np.abs(V - V_o)) < tol * max(1.0, np.max(np.abs(V_o)))
    assert np.all(np.triu(V, 1) == 0) and np.all(np.diag(V) == 1)
    assert np.all(np.tril(T, -1) == 0)
    G = V.T @ V
    M = T.T @ G @ T - T - T.T
    assert np.linalg.norm(M) * np.linalg.norm(V, 2) ** 2 < 1e-12
    R = Y - V @ (T.T @ (V.T @ Y))
    assert np.linalg.norm(np.tril(R, -1)) <= 1e-13 * np.linalg.norm(Y)


@pytest.mark.parametrize("m,b", [(1, 1), (16, 16), (17, 15), (33, 17), (64, 31), (64, 64),
                                 (65, 33), (129, 16), (128, 63), (513, 16), (257, 32),
                                 (640, 47), (3001, 49), (9000, 64), (20000, 64), (40000, 32)])
def test_panel_at_block_and_grid_edges(m, b):
    say(f"panel blocks m={m} b={b}")
    # cond(Y) = 100: 1e4 eps covers 100 cond(Y) u.
    _check(W.random_graded(m, b, np.float64, 100 + m + b, decay=1e-2), 1e4 * 2.3e-16)


@pytest.mark.parametrize("m,b,drop", [(300, 64, 5), (300, 64, 16), (300, 64, 37), (5000, 48, 15),
                                      (5000, 48, 17)])
def test_panel_sweep_ends_inside_a_block(m, b, drop):
    # Columns from `drop` on are the first one plus a remainder of 1e-3: their
    # norms cancel when column 0 is removed, so the sweep ends at `drop` (and
    # goes on there); cond(Y) is about 1e4.
    say(f"panel sweep m={m} b={b} drop={drop}")
    Y = W.random_dense(m, b, np.float64, 7 + drop)
    Y[:, drop:] = Y[:, :1] + 1e-3 * Y[:, drop:]
    _check(np.asfortranarray(Y), 100 * 1e4 * 2.3e-16)


@pytest.mark.parametrize("m,b,zero", [(3000, 64, [11]), (3000, 48, [12, 13]), (9000, 64, [0, 14]),
                                      (200, 64, [15, 16, 63]), (5000, 32, [0, 11, 31]),
                                      (5000, 16, [3, 15])])
def test_panel_columns_zero_below_the_diagonal(m, b, zero):
    # H = I for them, in whatever place of a 16-column block they stand.
    say(f"panel zero columns m={m} b={b} zero={zero}")
    Y = W.random_graded(m, b, np.float64, 31 + m + b, decay=1e-2)
    Y[:, zero] = 0.0
    _check(Y, 1e4 * 2.3e-16)


@pytest.mark.parametrize("rows", [12, 16])
def test_run_on_a_matrix_of_few_nonzero_rows(rows):
    # The first panel's columns from `rows` on are zero below the diagonal.
    say(f"run few rows {rows}")
    A = np.zeros((700, 400), order="F")
    A[:rows] = W.random_dense(rows, 400, np.float64, rows)
    ref = oracle.hbarrf(A, 1e-8, 48, 5)
    with rrf.Plan(torch.float64, 700, 400, 48) as p:
        Q, B, k = p.run(to_dev(A), 1e-8, 48, 5)
        Q, B = to_host(Q), to_host(B)
    assert k == ref.k
    assert np.linalg.norm(Q.T @ Q - np.eye(k)) < 1e-12
    assert np.linalg.norm(A - Q @ B) < 1e-13 * np.linalg.norm(A)

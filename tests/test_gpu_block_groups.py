"""Blocks of at most 32 columns run several to a sub-block: the stop test must
still end the run at the right block, with the trace, T and the results of
single blocks."""

import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
import paper_2608_28941_amd as rrf
from gpu_util import say, to_dev, to_host

pytestmark = pytest.mark.gpu


# 1100 x 900 doubles are above 4 MiB (up to 64 columns), 300 x 200 below.
@pytest.mark.parametrize("mode", [rrf.RRF_STOP_TRAILING, rrf.RRF_STOP_SUBTRACT])
@pytest.mark.parametrize("m,n,b", [(300, 200, 16), (300, 200, 10), (1100, 900, 16),
                                   (1100, 900, 32), (1100, 900, 24), (1100, 900, 20)])
def test_stop_inside_a_sub_block(m, n, b, mode):
    # Tolerances that end the run after 1, 2, 3, ... blocks: the geometric mean
    # of the residuals after consecutive blocks.
    w = W.scaled("tiny_fp64_500x300", m, n)
    A = W.build_matrix(w)
    ref = oracle.hbarrf(A, 1e-4, b, w.sketch_seed)
    E = np.asarray([t[1] for t in ref.trace])
    E0 = float(np.sum(A * A))
    with rrf.Plan(torch.float64, m, n, b) as p:
        p.set_stop_mode(mode)
        for nb in (1, 2, 3, 4, min(6, len(E))):
            prev = E0 if nb == 1 else E[nb - 2]
            tol = float(np.sqrt(np.sqrt(prev * E[nb - 1]) / E0))
            say(f"block group m={m} n={n} b={b} mode={mode} blocks={nb}")
            Q, B, k = p.run(to_dev(A), tol, b, w.sketch_seed)
            tr = p.trace()
            V, T, tau = p.reflectors(m, k)
            Q, B, V, T = to_host(Q), to_host(B), to_host(V), to_host(T)
            assert k == nb * b and tr["nblocks"] == nb
            # The trace's norms: binary64 sums of at most m n squares.
            assert np.allclose(tr["E_trail"], E[:nb], rtol=1e-9, atol=0)
            assert np.allclose(tr["E_sub"], E[:nb], rtol=1e-9, atol=1e-13 * E0)
            assert np.linalg.norm(Q.T @ Q - np.eye(k)) < 1e-12
            assert np.linalg.norm(B - Q.T @ A) < 1e-12 * np.sqrt(E0)
            # Each block's own reflector, from V and the first b rows of T.
            X = A.copy()
            for i in range(nb):
                c = slice(i * b, (i + 1) * b)
                Vi, Ti = V[:, c], np.triu(T[:b, c])
                M = Ti.T @ (Vi.T @ Vi) @ Ti - Ti - Ti.T
                assert np.linalg.norm(M) * np.linalg.norm(Vi, 2) ** 2 < 1e-12
                X = X - Vi @ (Ti.T @ (Vi.T @ X))
            assert np.linalg.norm(X[:k] - B) < 1e-11 * np.sqrt(E0)


@pytest.mark.parametrize("b,kmax", [(16, 50), (32, 96), (24, 100), (7, 30)])
def test_rank_cap_inside_a_sub_block(b, kmax):
    w = W.scaled("tiny_fp64_500x300", 1100, 900)
    A = W.build_matrix(w)
    ref = oracle.hbarrf(A, 0.0, b, w.sketch_seed, k_max=kmax)
    with rrf.Plan(torch.float64, 1100, 900, b, k_max=kmax) as p:
        Q, B, k = p.run(to_dev(A), 0.0, b, w.sketch_seed)
        assert k == kmax and p.last_status == rrf._abi.RRF_WARN_KMAX
        assert p.trace()["nblocks"] == -(-kmax // b)
        # cond(A Omega_k) is about 10^(kmax / 30): well inside 1e-9.
        assert np.max(np.abs(to_host(Q) - ref.Q)) < 1e-9


@pytest.mark.parametrize("m,n,b", [(1100, 900, 16), (1100, 900, 24), (1500, 1400, 8)])
def test_early_stop_takes_at_most_32_columns(m, n, b):
    # A run that its first block ends: the first sample (the only one that is
    # not taken back as queued ahead; the panel beside the second one adds
    # 3 m 32^2 at most) holds at most 32 columns.
    say(f"early stop m={m} n={n} b={b}")
    A = W.random_dense(m, b - 3, np.float64, b) @ W.random_dense(b - 3, n, np.float64, b + 1)
    with rrf.Plan(torch.float64, m, n, b) as p:
        Q, B, k = p.run(to_dev(np.asfortranarray(A)), 1e-8, b, 3)
        sample = p.stage_stats()["sample"]["flops"]
        Q, B = to_host(Q), to_host(B)
    assert k == b
    assert sample <= 2.0 * m * n * 32 + 3.0 * m * 32 ** 2
    assert np.linalg.norm(A - Q @ B) < 1e-12 * np.linalg.norm(A)


@pytest.mark.parametrize("lookahead", ["1", "0"])
@pytest.mark.parametrize("b", [8, 16, 24, 32])
def test_sub_blocks_widen_on_the_way(monkeypatch, b, lookahead):
    # A slow decay: 32 columns at first, 64 once the stop is known to be far.
    monkeypatch.setenv("RRF_LOOKAHEAD", lookahead)
    say(f"sub-blocks widen b={b} lookahead={lookahead}")
    m, n, tol = 1100, 900, 3e-3
    A = W.random_graded(m, n, np.float64, 17)
    ref = oracle.hbarrf(A, tol, b, 9)
    with rrf.Plan(torch.float64, m, n, b) as p:
        Q, B, k = p.run(to_dev(A), tol, b, 9)
        tr, updates = p.trace(), p.stage_stats()["update"]["launches"]
        V, T, _ = p.reflectors(m, k)
        Q, B, V, T = to_host(Q), to_host(B), to_host(V), to_host(T)
    assert k == ref.k and tr["nblocks"] == len(ref.trace)
    # At most one pass per min(4 blocks, 64 columns), and the first 32-column
    # ones: 8 with look-ahead, 2 without.
    cols = min(4, 64 // b) * b
    assert updates <= 1 + -(-k // cols) + (8 if lookahead == "1" else 2)
    assert np.allclose(tr["E_trail"], [t[1] for t in ref.trace], rtol=1e-9, atol=0)
    # cond(A Omega_k) is at most about 1e4 here.
    assert np.max(np.abs(Q - ref.Q)) < 1e3 * 1e4 * 2.3e-16
    assert np.linalg.norm(B - Q.T @ A) < 1e-12 * np.linalg.norm(A)
    for i in range(0, k, b):
        c = slice(i, min(i + b, k))
        w = c.stop - c.start
        Vi, Ti = V[:, c], np.triu(T[:w, c])
        assert np.linalg.norm(Ti.T @ (Vi.T @ Vi) @ Ti - Ti - Ti.T) < 1e-11

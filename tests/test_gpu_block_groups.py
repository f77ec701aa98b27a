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

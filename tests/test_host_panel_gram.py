"""The Gram panel's own source on the CPU (host_panel_gram.cpp): its lanes run
as fibers and LDS starts as NaNs, so a value that is read before it is written
shows in the results."""

import os
import re
import shutil
import subprocess

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_28941_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
U = np.finfo(np.float64).eps / 2


@pytest.fixture(scope="module")
def panel(tmp_path_factory):
    """panel(Y, G, rt) -> V, T, tau of the compiled body; panel.exchanges: the
    grid exchanges of the last call (G > 1)."""
    clang = next((c for c in (os.path.join(ROCM, "llvm", "bin", "clang++"),
                              shutil.which("amdclang++")) if c and os.path.exists(c)), None)
    if clang is None:
        pytest.skip("clang++ not available")
    d = tmp_path_factory.mktemp("host_panel")
    (d / "pkg" / "csrc").mkdir(parents=True)
    (d / "include").mkdir()
    shutil.copy(os.path.join(ROOT, "include", "rrf.h"), d / "include")
    for h in ("panel_gram_body.h", "lanes.h", "mfma.h", "xchg.h", "rrf_internal.h"):
        text = open(os.path.join(CSRC, h)).read()
        # The one inline statement names a vector register: any register here.
        (d / "pkg" / "csrc" / h).write_text(re.sub(r'"\+v"', '"+r"', text))
    exe = str(d / "panel")
    r = subprocess.run([clang, "-std=c++17", "-O2", "-ffp-contract=off", "-Wno-psabi",
                        "-mavx2", "-mfma", "-D__HIP_PLATFORM_AMD__", "-I",
                        os.path.join(ROCM, "include"), "-I", str(d / "pkg" / "csrc"), "-I",
                        os.path.join(ROOT, "tests"),
                        os.path.join(ROOT, "tests", "host_panel_gram.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def go(Y, G=1, rt=1, fill=0xFF):
        m, b = Y.shape
        bp = 16 if b <= 16 else 32 if b <= 32 else 64
        fin, fout = str(d / "in"), str(d / "out")
        np.ascontiguousarray(Y.T).tofile(fin)
        r = subprocess.run([exe, str(bp), str(rt), str(G), str(b), str(m), str(fill), fin, fout],
                           timeout=120)
        assert r.returncode == 0
        o = np.fromfile(fout)
        assert o[-1] == 0          # no wait gave up
        go.exchanges = int(o[-2])
        return (o[:m * b].reshape(b, m).T, o[m * b:m * b + b * b].reshape(b, b).T,
                o[m * b + b * b:m * b + b * b + b])

    return go


def _check(Y, V, T, tau):
    # cond of the panels below is at most 1e3, and 1e4 cond u covers the
    # factor that the tests of the stages state for 100 cond u and b columns.
    V_o, tau_o = oracle.geqr2(Y)
    assert np.all(np.isfinite(V)) and np.all(np.isfinite(T))
    assert np.max(np.abs(tau - tau_o)) < 1e4 * 1e3 * U
    assert np.max(np.abs(V - V_o)) < 1e4 * 1e3 * U
    assert np.all(np.triu(V, 1) == 0) and np.all(np.diag(V) == 1)
    assert np.all(np.tril(T, -1) == 0)
    assert np.linalg.norm(T.T @ (V.T @ V) @ T - T - T.T) < 1e-12


@pytest.mark.parametrize("m,b,G,rt", [(64, 64, 1, 1), (40, 16, 1, 1), (60, 31, 1, 1),
                                      (100, 49, 2, 1), (128, 64, 1, 2)])
def test_body_matches_oracle(panel, m, b, G, rt):
    Y = np.random.default_rng(m + b).standard_normal((m, b))
    _check(Y, *panel(Y, G, rt))


@pytest.mark.parametrize("m,b,G,zero", [
    (100, 64, 2, [0]), (100, 64, 2, [11]), (100, 48, 2, [12, 13]), (64, 64, 1, [14, 15, 16]),
    (100, 64, 2, [31, 63]), (60, 32, 1, [0, 5, 20]), (50, 16, 1, [3, 15])])
def test_columns_zero_below_the_diagonal(panel, m, b, G, zero):
    # H = I for them: nothing of R^-T or V^-1 is formed, and nothing may be read.
    Y = np.random.default_rng(7 * m + b).standard_normal((m, b))
    Y[:, zero] = 0.0
    V, T, tau = panel(Y, G)
    _check(Y, V, T, tau)
    assert np.all(tau[zero] == 0) and np.all(V[:, zero] == np.eye(m)[:, zero])


@pytest.mark.parametrize("rows", [1, 12, 16, 17])
def test_panel_of_few_nonzero_rows(panel, rows):
    # Every column from `rows` on is zero below the diagonal.
    Y = np.random.default_rng(rows).standard_normal((90, 48))
    Y[rows:] = 0.0
    V, T, tau = panel(Y, 2)
    _check(Y, V, T, tau)
    assert np.all(tau[rows:] == 0)


@pytest.mark.parametrize("cols", [slice(None), slice(20, None), slice(None, None, 2)])
@pytest.mark.parametrize("e", [-515, -520, -525])
def test_tiny_columns(panel, e, cols):
    # Norms whose squares are subnormal: the reciprocal of the square overflows,
    # which must neither reach a result nor end the sweep at every column.
    Y = np.random.default_rng(40).standard_normal((100, 40))
    tau_o = oracle.geqr2(Y)[1]
    S = Y.copy()
    S[:, cols] = np.ldexp(S[:, cols], e)
    panel(Y, 2)
    sweeps = panel.exchanges
    V, T, tau = panel(S, 2)
    assert panel.exchanges <= sweeps + 1
    assert np.all(np.isfinite(V)) and np.all(np.isfinite(T))
    # A scale changes no tau.  A square of about 2^(2 e) is rounded to 2^-1074:
    # the norms' relative errors are about 2^(-1074 - 2 e), and 1e3 covers their
    # growth over 40 columns (as 1e4 above does for u).
    tol = 1e3 * 2.0 ** (-1074 - 2 * e) + 1e4 * U
    assert np.max(np.abs(tau - tau_o)) < tol
    assert np.linalg.norm(T.T @ (V.T @ V) @ T - T - T.T) < 10 * tol

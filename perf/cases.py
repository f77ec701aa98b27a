"""Workloads by which the speed of this library is followed.

Each case is one call, or one run, that a user's program makes through the
package's public entry points: whole range-finder runs (small, ordinary,
large; tall, wide and ragged; adaptive, fixed rank, power iterations, spectral
stop; both dtypes) and the stage calls a program uses on its own (subspace
map, panel QR, block reflector, sketch).

``exact`` restates each computation in float64 torch: Alg. 2 block by block
with LAPACK's geqrf for the panels and the plain compact-WY algebra for
everything else, with the Gaussian sketch from numpy's Philox words and
libm's log, cos and sin.

The float32 runs take inputs whose noise is well above float32's rounding: a
reflector's sign follows the sign of one entry of its column, and where that
entry is below the rounding error two correct results differ in the signs of
all later columns.  At a level l of the last directions about k 5 u / l of the
runs would meet such an entry (30 % at the noise of 1e-4 that the benchmark's
4096 x 11008 input has, 0.5 % here); the sizes are the benchmark's.
"""

import math

import numpy as np
import torch

import paper_2608_28941_amd as rrf

_DT = {"f32": torch.float32, "f64": torch.float64}
_DEV = "cuda"


def listed():
    """The workloads, smallest calls to the largest."""
    return [
        # Latency: a small dense matrix brought to four digits.
        dict(name="run_tiny_f64", op="run", m=500, n=300, dtype="f64", b=16, tol=1e-4,
             kmax=0, rank=300, law="pow10", decay=30.0, noise=0.0, power=0, stop="trailing",
             k=144),
        # Odd sizes and a ragged last block, no alignment anywhere, the
        # spectral-norm stop.
        dict(name="run_ragged_spectral_f64", op="run", m=3001, n=1733, dtype="f64", b=48,
             tol=1e-3, kmax=0, rank=500, law="pow10", decay=100.0, noise=1e-6, power=0,
             stop="spectral", k=336),
        # Slow decay: one power iteration to a fixed rank, the shape of an MLP
        # gradient of a smaller layer.
        dict(name="run_power_f32", op="run", m=2048, n=5461, dtype="f32", b=32, tol=0.0,
             kmax=256, rank=1024, law="ipow", decay=0.5, noise=1e-3, power=1,
             stop="trailing", k=256),
        # The optimiser's low-rank refresh of an MLP gradient, transposed
        # orientation, fixed rank 512 in blocks of 128.
        dict(name="run_fixed_f32", op="run", m=11008, n=4096, dtype="f32", b=128, tol=0.0,
             kmax=512, rank=1024, law="exp", decay=300.0, noise=1e-3, power=0,
             stop="trailing", k=512),
        # Gradient-shaped square matrix whose noise must be followed far down:
        # many narrow blocks.
        dict(name="run_galore_f32", op="run", m=4096, n=4096, dtype="f32", b=32, tol=0.086,
             kmax=0, rank=512, law="ipow", decay=1.5, noise=1e-2, power=0, stop="trailing",
             k=3424),
        # Wide gradient of an MLP layer.
        dict(name="run_mlp_f32", op="run", m=4096, n=11008, dtype="f32", b=64, tol=0.1,
             kmax=0, rank=256, law="exp", decay=40.0, noise=1e-2, power=0, stop="trailing",
             k=1856),
        # Tall and skinny, to eight digits.
        dict(name="run_tall_f64", op="run", m=131072, n=2048, dtype="f64", b=32, tol=1e-8,
             kmax=0, rank=200, law="flat", decay=20.0, noise=1e-10, power=0, stop="trailing",
             k=224),
        # The headline size.
        dict(name="run_square_f64", op="run", m=16384, n=16384, dtype="f64", b=64, tol=1e-6,
             kmax=0, rank=1024, law="pow10", decay=128.0, noise=1e-8, power=0,
             stop="trailing", k=960),
        # An optimiser state carried from one basis to the next.
        dict(name="map_f32", op="map", m=4096, n=11008, dtype="f32", r_old=448, r_new=512),
        # One panel on its own.
        dict(name="panel_f64", op="panel", m=16384, dtype="f64", b=64, decay=1e-2),
        # One block reflector on a gradient, Q^T X.
        dict(name="reflect_f32", op="reflect", m=4096, n=11008, dtype="f32", b=64,
             trans=True),
        # A Gaussian sketch on its own.
        dict(name="sketch_f32", op="sketch", n=11008, dtype="f32", ncols=512, col0=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    op = rng.choice(["run", "run", "run", "run", "map", "panel", "reflect", "sketch"])
    dtype = rng.choice(["f32", "f64"])
    if op == "map":
        return dict(op=op, m=_log_int(rng, 256, 16384), n=_log_int(rng, 64, 16384),
                    dtype=dtype, r_old=_log_int(rng, 16, 1024),
                    r_new=_log_int(rng, 16, 1024))
    if op == "panel":
        b = rng.choice([8, 16, 24, 32, 48, 64, rng.randint(1, 64)])
        return dict(op=op, m=_log_int(rng, 128, 131072), dtype=dtype, b=b,
                    decay=rng.choice([1.0, 1e-2, 1e-4]))
    if op == "reflect":
        b = rng.choice([8, 16, 32, 64, rng.randint(1, 64)])
        return dict(op=op, m=_log_int(rng, 128, 16384), n=_log_int(rng, 16, 16384),
                    dtype=dtype, b=b, trans=rng.random() < 0.5)
    if op == "sketch":
        return dict(op=op, n=_log_int(rng, 64, 131072), dtype=dtype,
                    ncols=rng.choice([16, 32, 64, 128, 256, rng.randint(1, 512)]),
                    col0=rng.randint(0, 4096))
    # Whole runs: up to 16384 a side and 2^27 elements (f32: 2^28), rank such
    # that the work stays below the largest listed case.
    m = _log_int(rng, 300, 16384)
    n = _log_int(rng, 300, 16384)
    while m * n > (1 << 27 if dtype == "f64" else 1 << 28):
        m, n = max(300, m // 2), max(300, n // 2)
    b = rng.choice([16, 24, 32, 48, 64, 96, 128])
    k = min(_log_int(rng, 32, 1024), min(m, n) // 2)
    nblk = max(1, round(k / b))
    kind = rng.random()
    if kind < 0.15:
        # Power iteration on a slowly decaying spectrum, fixed rank.
        k = min(k, 512)
        return dict(op=op, m=m, n=n, dtype=dtype, b=min(b, 64), tol=0.0, kmax=k,
                    rank=min(2 * k, min(m, n)), law="ipow", decay=0.5, noise=1e-3, power=1,
                    stop="trailing", k=k)
    if kind < 0.45:
        # Fixed rank, not always a multiple of the block.
        k = min(k if rng.random() < 0.5 else nblk * b, min(m, n) // 2)
        return dict(op=op, m=m, n=n, dtype=dtype, b=b, tol=0.0, kmax=k,
                    rank=min(2 * k, min(m, n)), law="exp", decay=0.4 * k + 4.0,
                    noise=1e-3, power=0, stop="trailing", k=k)
    # To a tolerance: exponential decay that reaches it near rank k.
    digits = rng.choice([1.0, 1.5]) if dtype == "f32" else rng.choice([2, 3, 4, 6])
    k = max(k, 16)
    return dict(op=op, m=m, n=n, dtype=dtype, b=b, tol=10.0 ** -digits, kmax=0,
                rank=min(2 * k + 16, min(m, n)), law="pow10", decay=k / (1.25 * digits),
                noise=10.0 ** (-digits - 2), power=0,
                stop="spectral" if rng.random() < 0.2 else "trailing", k=k)


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------

def _spectrum(law, decay, r):
    i = torch.arange(r, dtype=torch.float64, device=_DEV)
    if law == "pow10":
        return 10.0 ** (-i / decay)
    if law == "exp":
        return torch.exp(-i / decay)
    if law == "ipow":
        return (i + 1.0) ** -decay
    if law == "flat":
        return torch.where(i < 50, torch.ones_like(i), 10.0 ** (-(i - 50.0) / decay))
    raise ValueError(law)


def _gen(seed, stream):
    return torch.Generator(device=_DEV).manual_seed((int(seed) * 1000003 + stream) % (1 << 62))


def _randn(rows, cols, seed, stream):
    return torch.randn(rows, cols, dtype=torch.float64, device=_DEV, generator=_gen(seed, stream))


def _matrix(case, seed):
    """G1 diag(s) G2^T + noise N, column-major, rounded once to the dtype."""
    m, n, r = case["m"], case["n"], case["rank"]
    g1 = _randn(r, m, seed, 1) / math.sqrt(m)
    g2 = _randn(n, r, seed, 2) / math.sqrt(n)
    at = (g2 * _spectrum(case["law"], case["decay"], r)) @ g1       # n x m = A^T
    if case["noise"]:
        at.add_(_randn(n, m, seed, 3), alpha=case["noise"] / math.sqrt(max(m, n)))
    return at.to(_DT[case["dtype"]]).t()


def _ortho(rows, cols, seed, stream):
    """cols orthonormal columns (column-major, float64): Cholesky QR twice."""
    qt = _randn(cols, rows, seed, stream) / math.sqrt(rows)
    for _ in range(2):
        qt = torch.linalg.solve_triangular(torch.linalg.cholesky(qt @ qt.t()), qt, upper=False)
    return qt.t()


def _colmajor(t):
    return t.t().contiguous().t()


def _sketch_seed(seed):
    return (int(seed) * 7919 + 17) & 0x7FFFFFFFFFFFFFFF


def _panel(case, seed):
    """m x b with singular values graded from 1 to ``decay``, as sampled
    panels have."""
    m, b = case["m"], case["b"]
    y = _randn(b, m, seed, 11)
    s = torch.logspace(0.0, math.log10(case["decay"]), b, dtype=torch.float64, device=_DEV)
    mix = _randn(b, b, seed, 12) / math.sqrt(b)
    return ((mix * s) @ y / math.sqrt(m)).to(_DT[case["dtype"]]).t()


def _factor(y):
    """Householder QR of a float64 panel: V (unit lower trapezoidal), T with
    H_0 ... H_{b-1} = I - V T V^T, tau."""
    b = y.shape[1]
    a, tau = torch.geqrf(y.cpu())
    v = a.tril(-1)
    v.diagonal().fill_(1.0)
    t = torch.zeros(b, b, dtype=torch.float64)
    g = v.t() @ v
    for j in range(b):
        t[:j, j] = -tau[j] * (t[:j, :j] @ g[:j, j])
        t[j, j] = tau[j]
    return v.to(_DEV), t.to(_DEV), tau.to(_DEV)


def _reflector(case, seed):
    v, t, _ = _factor(_randn(case["b"], case["m"], seed, 21).t())
    dt = _DT[case["dtype"]]
    x = _randn(case["n"], case["m"], seed, 22).to(dt).t()
    return _colmajor(v.to(dt)), _colmajor(t.to(dt)), x


def _map_inputs(case, seed):
    dt = _DT[case["dtype"]]
    q_old = _ortho(case["m"], min(case["r_old"], case["m"]), seed, 31)
    q_new = _ortho(case["m"], min(case["r_new"], case["m"]), seed, 32)
    # Consecutive bases share most of their leading directions.
    c = min(q_old.shape[1], q_new.shape[1])
    mix = torch.cat([0.9 * q_old[:, :c] + 0.44 * q_new[:, :c], q_new[:, c:]], 1)
    mat = _randn(case["n"], q_old.shape[1], seed, 33).to(dt).t()
    return _colmajor(mix.to(dt)), _colmajor(q_old.to(dt)), mat


def prepare(case, seed):
    dt = _DT[case["dtype"]]
    op = case["op"]
    if op == "run":
        plan = rrf.Plan(dt, case["m"], case["n"], case["b"], k_max=case["kmax"])
        plan.set_power_iterations(case["power"])
        plan.set_stop_mode({"trailing": rrf.RRF_STOP_TRAILING,
                            "spectral": rrf.RRF_STOP_SPECTRAL}[case["stop"]])
        return dict(op=op, plan=plan, A=_matrix(case, seed), tol=case["tol"], b=case["b"],
                    seed=_sketch_seed(seed))
    if op == "map":
        q_new, q_old, mat = _map_inputs(case, seed)
        plan = rrf.Plan(dt, case["m"], case["n"], 64, k_max=64)
        return dict(op=op, plan=plan, args=(q_new, q_old, mat))
    if op == "panel":
        plan = rrf.Plan(dt, case["m"], case["b"], case["b"], k_max=case["b"])
        return dict(op=op, plan=plan, Y=_panel(case, seed))
    if op == "reflect":
        v, t, x = _reflector(case, seed)
        plan = rrf.Plan(dt, case["m"], case["n"], case["b"], k_max=case["b"])
        return dict(op=op, plan=plan, V=v, T=t, X=x, trans=case["trans"])
    return dict(op=op, dtype=dt, seed=_sketch_seed(seed), n=case["n"], col0=case["col0"],
                ncols=case["ncols"])


def run(state):
    op = state["op"]
    if op == "run":
        q, b, k = state["plan"].run(state["A"], state["tol"], state["b"], state["seed"])
        return {"Q": q, "B": b, "k": k}
    if op == "map":
        return state["plan"].subspace_map(*state["args"])
    if op == "panel":
        v, t, tau = state["plan"].panel_qr(state["Y"])
        return {"V": v, "T": t, "tau": tau}
    if op == "reflect":
        # In place, as the stage works: X stays of the same size, since the
        # reflector is orthogonal.
        return state["plan"].apply_block_reflector(state["V"], state["T"], state["X"],
                                                   trans=state["trans"])
    return rrf.sketch(state["dtype"], state["seed"], state["n"], state["col0"],
                      state["ncols"])


def work(case):
    e = 4 if case["dtype"] == "f32" else 8
    op = case["op"]
    if op == "run":
        m, n, k, b = case["m"], case["n"], case["k"], case["b"]
        # Sample, V^T B and the update over the trailing rows of each block
        # (6 m_i n b, and 4 m_i n b more per power iteration), explicit Q;
        # A read, Q and B written.
        fl = 0.0
        for i in range(0, k, b):
            w = min(b, k - i)
            fl += (6.0 + 4.0 * case["power"]) * (m - i) * n * w
        fl += 2.0 * m * k * k - 2.0 * k ** 3 / 3.0
        return {"bytes": float(e) * (m * n + m * k + k * n), "flops": fl}
    if op == "map":
        m, n, r0, r1 = case["m"], case["n"], case["r_old"], case["r_new"]
        r0, r1 = min(r0, m), min(r1, m)
        return {"bytes": float(e) * (m * (r0 + r1) + r0 * n + r1 * n),
                "flops": 2.0 * m * r0 * r1 + 2.0 * r0 * r1 * n}
    if op == "panel":
        m, b = case["m"], case["b"]
        return {"bytes": float(e) * (2 * m * b + b * b + b),
                "flops": 3.0 * m * b * b}
    if op == "reflect":
        m, n, b = case["m"], case["n"], case["b"]
        return {"bytes": float(e) * (2 * m * n + m * b + b * b),
                "flops": 4.0 * m * n * b + 1.0 * n * b * b}
    # About 25 multiply-adds per Gaussian after the Philox rounds.
    return {"bytes": float(e) * case["n"] * case["ncols"],
            "flops": 50.0 * case["n"] * case["ncols"]}


def _level(case):
    """The smallest singular value, relative to the largest, that the basis
    resolves: Q's last columns carry the rounding errors divided by it."""
    i = float(case["k"] if case["kmax"] else -(-case["k"] // case["b"]) * case["b"])
    d = case["decay"]
    s = {"pow10": lambda: 10.0 ** (-i / d), "exp": lambda: math.exp(-i / d),
         "ipow": lambda: (i + 1.0) ** -d,
         "flat": lambda: 10.0 ** (-max(0.0, i - 50.0) / d)}[case["law"]]()
    return max(s, case["noise"])


def tolerance(case):
    # About four times the distance from ``exact`` (two correct results also
    # differ by their two errors): runs measured 1e-11 (tiny, level 1.6e-5),
    # 4.6e-9 (square, 1e-8), 6e-6 (tall, 1e-10), f32 1e-6 to 5e-6 and 2e-4
    # at level 1e-4; panels 5e-12 at decay 1e-2, 1e-10 at 1e-4; map 4e-7 and
    # reflector 2.3e-7 in f32, which grow with the root of the rows.
    f32 = case["dtype"] == "f32"
    op = case["op"]
    if op == "sketch":
        return "exact"
    if op == "run":
        rel = (2e-5 + 1.5e-7 / _level(case)) if f32 else (1e-11 + 2e-15 / _level(case))
        rel = min(rel, 0.02)
    elif op == "panel":
        rel = (1.5e-7 if f32 else 0.0) + 1e-13 / case["decay"]
    elif op == "map":
        rel = 4e-6 if f32 else 2e-14
    else:
        rel = 2e-6 if f32 else 4e-15
    return {"rel": rel, "max": min(0.9, 500.0 * rel)}


# ---------------------------------------------------------------------------
# The same results in float64.
# ---------------------------------------------------------------------------

def _sketch64(seed, n, col0, ncols):
    """Gaussian columns: Philox4x64-10 words with counter (row/4, column, 0, 0)
    and key (seed, 0), Box-Muller on the word pairs."""
    nb = (n + 3) // 4
    words = np.empty((ncols, nb, 4), dtype=np.uint64)
    for j in range(ncols):
        bits = np.random.Philox(key=seed, counter=((col0 + j << 64) - 1) % (1 << 256))
        words[j] = bits.random_raw(4 * nb).reshape(nb, 4)
    out = np.empty((ncols, nb, 4))
    for a in (0, 2):
        u1 = ((words[:, :, a] >> np.uint64(11)) + np.uint64(1)).astype(np.float64) * 2.0 ** -53
        u2 = (words[:, :, a + 1] >> np.uint64(11)).astype(np.float64) * 2.0 ** -53
        r = np.sqrt(-2.0 * np.log(u1))
        out[:, :, a] = r * np.cos(2.0 * np.pi * u2)
        out[:, :, a + 1] = r * np.sin(2.0 * np.pi * u2)
    return torch.from_numpy(out.reshape(ncols, 4 * nb)[:, :n].copy()).t()


def _spectral_estimate(bt, y):
    """Largest eigenvalue of (Z^T Z, Y^T Y), Z = Bt^T Y."""
    q, _ = torch.linalg.qr(y.cpu())
    return float(torch.linalg.matrix_norm((bt.t() @ q.to(_DEV)).cpu(), 2)) ** 2


def _range_finder(case, seed):
    dt = _DT[case["dtype"]]
    bt = _matrix(case, seed).double().contiguous()
    m, n, b = case["m"], case["n"], case["b"]
    cap = min(m, n, case["kmax"] or min(m, n))
    e0 = float((bt * bt).sum())
    sigma2 = case["tol"] ** 2 * e0
    sk = _sketch_seed(seed)

    def omega(k, w):
        return _sketch64(sk, n, k, w).to(dt).double().to(_DEV)

    fac, k, stop = [], 0, e0 <= sigma2
    while not stop and k < cap:
        w = min(b, cap - k)
        y = bt[k:] @ omega(k, w)
        for _ in range(case["power"]):
            y = bt[k:] @ (bt[k:].t() @ y) / e0
        v, t, _ = _factor(y)
        bt[k:] -= v @ (t.t() @ (v.t() @ bt[k:]))
        fac.append((k, v, t))
        k += w
        e = float((bt[k:] * bt[k:]).sum())
        if case["stop"] == "spectral" and k < cap:
            e = _spectral_estimate(bt[k:], bt[k:] @ omega(k, min(b, 64, cap - k)))
        stop = e <= sigma2
    q = torch.zeros(m, k, dtype=torch.float64, device=_DEV)
    q.diagonal().fill_(1.0)
    for k0, v, t in reversed(fac):
        q[k0:, k0:] -= v @ (t @ (v.t() @ q[k0:, k0:]))
    # Where the last columns of Q come from directions ten digits down, float64
    # does not determine them to more digits than the library's own float64:
    # such a Q has no better value to be compared with (B has: it is small
    # there).
    q = _colmajor(q) if case["dtype"] == "f32" or _level(case) > 1e-9 else None
    return {"Q": q, "B": _colmajor(bt[:k].clone()), "k": k}


def exact(case, seed):
    op = case["op"]
    if op == "run":
        return _range_finder(case, seed)
    if op == "map":
        q_new, q_old, mat = (t.double() for t in _map_inputs(case, seed))
        return _colmajor((q_new.t().contiguous() @ q_old) @ mat)
    if op == "panel":
        v, t, tau = _factor(_panel(case, seed).double())
        return {"V": _colmajor(v), "T": _colmajor(t), "tau": tau}
    if op == "reflect":
        v, t, x = (a.double() for a in _reflector(case, seed))
        t = t.t().contiguous() if case["trans"] else t
        return _colmajor(x - v @ (t @ (v.t().contiguous() @ x)))
    return _colmajor(_sketch64(_sketch_seed(seed), case["n"], case["col0"], case["ncols"])
                     .to(_DEV))

"""The subspace map at the edges of its tiles: rows and columns one off a tile,
a contracted index that is not whole packs or chunks, unaligned leading
dimensions, and sizes on both sides of the 128-row tiles."""

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
import paper_2608_28941_amd as rrf
from gpu_util import say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("m,r_new,r_old,n,pad", [(33, 1, 1, 1, 0), (64, 63, 65, 64, 1),
                                                 (129, 65, 127, 63, 3), (1000, 128, 129, 1030, 0),
                                                 (4100, 300, 260, 4097, 2), (515, 17, 130, 9000, 4)])
def test_map_at_tile_edges(dtype, m, r_new, r_old, n, pad):
    say(f"map tiles {np.dtype(dtype).name} m={m} r_new={r_new} r_old={r_old} n={n} pad={pad}")
    qn = W.random_dense(m, r_new, dtype, 1) / np.sqrt(m)
    qo = W.random_dense(m, r_old, dtype, 2) / np.sqrt(m)
    mm = W.random_dense(r_old, n, dtype, 3)
    qn, qo = (np.asfortranarray(x.astype(dtype)) for x in (qn, qo))

    def dev(x):
        # A column-major view with `pad` extra rows per column.
        big = torch.zeros((x.shape[1], x.shape[0] + pad), dtype=torch.from_numpy(x[:1, :1].copy()).dtype,
                          device="cuda")
        big[:, :x.shape[0]] = to_dev(x).t()
        return big.t()[:x.shape[0]]

    tdt = torch.float64 if dtype == np.float64 else torch.float32
    with rrf.Plan(tdt, m, n, 64, k_max=64) as p:
        got = to_host(p.subspace_map(dev(qn), dev(qo), dev(mm)))
    f = np.float64
    ref = (qn.astype(f).T @ qo.astype(f)) @ mm.astype(f)
    # Each product of length L errs by at most L u sum |a||b|; with entries of
    # order 1/sqrt(m) and 1 that is below 8 sqrt((m + r_old) r_old) u max|M|.
    tol = 8 * np.sqrt((m + r_old) * r_old) * np.finfo(dtype).eps * np.max(np.abs(mm))
    assert np.max(np.abs(got - ref)) < tol

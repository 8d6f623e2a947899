"""The segmented BFS of narrow bands against scipy's shortest paths.

Distances are integers: every comparison is exact.  Bands of half-width 1 to
8, segment edges (2,048 rows, a last segment shorter than the boundary), holes
that force paths back across a cut, a snake that crosses every cut eight
times, and one whose levels in a segment span more than the fill's range, so
that the queue kernels take the sweep."""

import numpy as np
import pytest
import scipy.sparse as sp
from scipy.sparse import csgraph

import workloads as W

pytestmark = pytest.mark.gpu


def _pattern(n, dists, density, seed, keep_path=False):
    rng = np.random.default_rng(seed)
    a = sp.csr_matrix((n, n))
    for d in dists:
        v = (rng.uniform(size=n - d) < density).astype(float)
        if keep_path and d == dists[0]:
            v[:] = 1.0
        a = a + sp.diags([-v, -v], [d, -d], shape=(n, n))
    return W.CSR.from_scipy(sp.csr_matrix(a) + sp.identity(n) * 20.0)


def _snake(n):
    """Eight chains of stride 8, joined at alternating ends: one path of n rows."""
    i = np.arange(n - 8)
    a = sp.coo_matrix((-np.ones(n - 8), (i, i + 8)), shape=(n, n)).tolil()
    for r in range(7):
        last = n - 8 + np.arange(8)
        if r % 2 == 0:
            u = [x for x in last if x % 8 == r][0]
            v = [x for x in last if x % 8 == r + 1][0]
        else:
            u, v = r, r + 1
        a[min(u, v), max(u, v)] = -1.0
    a = a.tocsr()
    return W.CSR.from_scipy(a + a.T + sp.identity(n) * 20.0)


CASES = [(f"full_w{w}", lambda w=w: _pattern(8192 + 17 * w, list(range(1, w + 1)), 1.0, w)) for w in range(1, 9)] + [
    ("n8192", lambda: _pattern(8192, [1, 2, 3], 1.0, 1)),
    ("last_segment_3_rows", lambda: _pattern(8195, [1, 5, 8], 1.0, 2)),
    ("last_segment_9_rows", lambda: _pattern(10249, [1, 8], 0.9, 3, keep_path=True)),
    ("density_80", lambda: _pattern(30000, list(range(1, 9)), 0.8, 4)),
    ("density_40", lambda: _pattern(30011, list(range(1, 9)), 0.4, 5)),
    ("density_25", lambda: _pattern(20000, list(range(1, 9)), 0.25, 6)),        # detours, perhaps not connected
    ("sparse_3_8", lambda: _pattern(16384, [3, 8], 0.97, 7)),
    ("disconnected", lambda: _pattern(9000, [2, 4, 8], 1.0, 8)),                 # even and odd rows
    ("snake", lambda: _snake(8192)),
    ("snake_long", lambda: _snake(40008)),                                       # beyond the fill's range
]


@pytest.mark.parametrize("name,gen", CASES, ids=[c[0] for c in CASES])
def test_distances(name, gen):
    from paper_2412_08059_amd import DeviceCSR, Solver
    a = gen()
    A = DeviceCSR.from_host(a)
    s = Solver(a.n, a.nnz)
    pat = abs(a.to_scipy())
    for src in (0, a.n - 1, a.n // 2 + 3, 2047, 2048):
        ref = csgraph.shortest_path(pat, method="D", unweighted=True, indices=src)
        ref = np.where(np.isinf(ref), -1, ref).astype(np.int64)
        st, dist, ecc, far = s.bfs(A, src)
        assert st == 0
        assert np.array_equal(dist.cpu().numpy(), ref), (name, src)
        assert ecc == ref.max()
        assert far == int(np.flatnonzero(ref == ref.max())[0])
    s.close()


@pytest.mark.parametrize("name", ["full_w8", "density_40", "density_25", "disconnected", "snake_long"])
def test_features_match_the_oracle(name):
    import oracle
    import torch
    from paper_2412_08059_amd import DeviceCSR, Solver
    a = dict(CASES)[name]()
    _, b = W.rhs(a, seed=1)
    s = Solver(a.n, a.nnz)
    st, f = s.features(DeviceCSR.from_host(a), torch.from_numpy(b).cuda())
    assert st == 0
    assert (f.pdiam, f.bfs_t, f.bfs_u, f.n_components) == oracle.pseudo_diameter(a)
    starts = [0, 5, a.n // 3]
    st, d = s.diameter_multi(DeviceCSR.from_host(a), starts, 0.9)
    assert st == 0
    want = oracle.diameter_multi(a, starts, 0.9)
    assert (d.pdiam, d.pdiam_multi, d.eff_diam, d.pairs, d.best_start) == want
    s.close()

"""The graph build at the edges of its row classes: block rows in decreasing
order, and the merged pull rows behind them (a bottom-up search reads nothing
else, so its parents, the highest frontier neighbours, show every entry's
place) against numpy and the oracle."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int64)).cuda()


# row lengths around the thread / wave / workgroup / radix classes and around
# one radix chunk; p = 3 puts the rows of a hub into three blocks
@pytest.mark.parametrize("p", [1, 3])
@pytest.mark.parametrize("length", [1, 2, 32, 33, 1023, 1024, 1025, 16384, 16385, 24577, 50000])
def test_rows_of_one_length(length, p):
    from paper_1208_5542_amd import csbfs
    rng = np.random.default_rng(length * 8 + p)
    n = 64 * p * 171
    R = n // p
    hubs = [5, n // 2, n - 1]
    src, dst = [], []
    for h in hubs:  # `length` entries of each hub in one block (duplicates where it is longer than R)
        lo = R * int(rng.integers(0, p))
        src.append(np.full(length, h))
        dst.append(lo + rng.integers(0, R, length))
    src.append(rng.integers(0, n, 2 * n))
    dst.append(rng.integers(0, n, 2 * n))
    src, dst = np.concatenate(src), np.concatenate(dst)
    g = csbfs.Graph(_dev(src), _dev(dst), n, p)
    a, b = np.r_[src, dst], np.r_[dst, src]
    for i in range(p):
        for j in range(p):
            rp, col = (x.cpu().numpy() for x in g.block(i, j))
            m = (a // R == j) & (b // R == i)
            u, v = a[m] - j * R, b[m] - i * R
            order = np.lexsort((-v, u))
            assert (rp == np.r_[0, np.cumsum(np.bincount(u, minlength=R))]).all(), (i, j)
            assert (col.astype(np.int64) == v[order]).all(), (i, j)
    adj = oracle.Adjacency(n, src, dst)
    V = oracle.directory(n, p, src, dst).reshape(-1)
    for root in hubs[:2]:
        ref = adj.alg3(p, V, root)
        for flags in (csbfs.FLAG_BOTTOM_UP_ONLY, 0):
            r = csbfs.Engine(g, flags=flags).bfs(root)
            assert (r.level.cpu().numpy() == ref.level).all(), flags
            assert (r.parent.cpu().numpy() == ref.parent).all(), flags


# builds that sort their entries (2^18 of them or more): counts around the
# rule and around a sort tile of 4096, id ranges whose keys end within a digit,
# and tuples that all lie in one row
@pytest.mark.parametrize("kind", ["uniform", "one_pair", "loops"])
@pytest.mark.parametrize("m,n,p", [((1 << 17) - 1, 64 * 40, 1), (1 << 17, 64 * 40, 1), ((1 << 17) + 1, 64 * 3 * 9, 3),
                                   ((1 << 17) + 2047, 1 << 16, 4), ((1 << 17) + 2049, (1 << 16) - 64, 1),
                                   (300007, 64 * 64 * 3, 64), (1 << 19, 64 * 7 * 500, 7)])
def test_sorted_builds(m, n, p, kind):
    from paper_1208_5542_amd import csbfs
    rng = np.random.default_rng(m + n)
    R = n // p
    if kind == "uniform":
        src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    elif kind == "one_pair":
        src, dst = np.full(m, n - 1), np.zeros(m, dtype=np.int64)
    else:
        src = rng.integers(n // 2, n // 2 + 3, m)
        dst = src.copy()
    g = csbfs.Graph(_dev(src), _dev(dst), n, p)
    a, b = np.r_[src, dst], np.r_[dst, src]
    block = (b // R) * p + a // R
    order = np.lexsort((-b, a, block))
    sizes = np.bincount(block, minlength=p * p)
    at = np.r_[0, np.cumsum(sizes)]
    a, b = a[order], b[order]
    for q in range(p * p):
        rp, col = (x.cpu().numpy() for x in g.block(q // p, q % p))
        u, v = a[at[q]:at[q + 1]] - (q % p) * R, b[at[q]:at[q + 1]] - (q // p) * R
        assert (rp == np.r_[0, np.cumsum(np.bincount(u, minlength=R))]).all(), q
        assert (col.astype(np.int64) == v).all(), q


@pytest.mark.parametrize("bad", [-1, 64 * 40, 1 << 33])
def test_sorted_build_refuses_ids_out_of_range(bad):
    from paper_1208_5542_amd import csbfs
    m, n = 1 << 17, 64 * 40
    for k in (0, 1):
        t = np.zeros((2, m), dtype=np.int64)
        t[k, m - 3] = bad
        with pytest.raises(csbfs.CsbfsError):
            csbfs.Graph(_dev(t[0]), _dev(t[1]), n, 1)

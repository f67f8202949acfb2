"""Bottom-up levels of batched searches on rows of every length class: the
lanes' own steps, the rows a wave reads side by side, and the long rows whole
workgroups read. Levels against the oracle; the entries read against the
counting rule (two ids, 16 steps of two, then steps of 64 until every missing
root is found)."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _read(row, fm, missing):
    got, e = 0, 0
    while e < len(row) and got != missing:
        step = 2 if e < 34 else 64
        for u in row[e:e + step]:
            got |= int(fm[u]) & missing
        e += min(step, len(row) - e)
    return e


@pytest.mark.parametrize("p", [1, 3])
@pytest.mark.parametrize("left", [1, 63, 64, 65, 257, 2047, 2048, 2049, 4097])
def test_bottom_up_rows(left, p):
    from paper_1208_5542_amd import csbfs
    n, d = 64 * 3 * 32, 34 + left  # hubs with `left` entries after the lane steps
    rng = np.random.default_rng(left * 8 + p)
    hubs = (n // 2, n // 3, 5)
    src, dst = [], []
    for k, h in enumerate(hubs):
        nb = rng.integers(0, n - 40, d)
        if k == 0:
            nb[-1] = 0  # only the row's last entry (lowest id) leads to root 0's component
            nb[:-1] += 1 + (nb[:-1] == 0)
        src += [np.full(d, h)]
        dst += [nb]
    # chains from the roots, so that the hubs are found late or not at all
    src += [np.array([n - 1, n - 2, n - 3, n - 5]), rng.integers(0, n - 40, 500)]
    dst += [np.array([n - 2, n - 3, 0, n - 6]), rng.integers(0, n - 40, 500)]
    src, dst = np.concatenate(src).astype(np.int64), np.concatenate(dst).astype(np.int64)
    roots = [n - 1, n - 5, int(dst[1]), int(dst[d + 2]), 5]
    g = csbfs.Graph(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), n, p)
    eng = csbfs.BatchEngine(g, max_roots=8, max_levels=64, flags=csbfs.FLAG_BOTTOM_UP_ONLY)
    r = eng.bfs(roots)
    torch.cuda.synchronize()
    adj = oracle.Adjacency(n, src, dst)
    ref = np.stack([adj.bfs(s) for s in roots])
    assert (r.level.cpu().numpy() == ref).all()
    rows = [[] for _ in range(n)]
    for a, b in zip(src.tolist(), dst.tolist()):
        rows[a].append(b)
        rows[b].append(a)
    rows = [sorted(x, reverse=True) for x in rows]
    for k in range(r.n_levels):
        fm = np.zeros(n, dtype=np.int64)
        vis = np.zeros(n, dtype=np.int64)
        active = 0
        for b in range(len(roots)):
            at = ref[b] == k
            active |= (1 << b) if at.any() else 0
            fm |= at.astype(np.int64) << b
            vis |= ((ref[b] >= 0) & (ref[b] <= k)).astype(np.int64) << b
        want = sum(_read(rows[v], fm, active & ~int(vis[v])) for v in range(n) if rows[v] and active & ~int(vis[v]))
        assert r.stats[k]["direction"] == 1 and r.stats[k]["edges"] == want, k


@pytest.mark.parametrize("n", [(1 << 20) - 64, 1 << 20, (1 << 20) + 64])
@pytest.mark.parametrize("dense", [False, True])
def test_bottom_up_through_the_frontier_bitmap(n, dense):
    """Sparse and wide union frontiers on either side of the sizes that look
    neighbours up in the frontier's bitmap: same levels, same entries read."""
    from paper_1208_5542_amd import csbfs
    rng = np.random.default_rng(n + dense)
    used = rng.choice(n, 120000 if dense else 3000, replace=False)
    hub = int(used[0])
    src = np.concatenate([used[rng.integers(0, used.size, 40000)], np.full(6000, hub), used if dense else used[:2]])
    dst = np.concatenate([used[rng.integers(0, used.size, 40000)], used[rng.integers(0, used.size, 6000)],
                          np.full(used.size if dense else 2, int(used[1]))])
    roots = [int(used[1]), hub, int(used[7]), int(dst[5])]
    g = csbfs.Graph(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), n, 1)
    r = csbfs.BatchEngine(g, max_roots=4, max_levels=64, flags=csbfs.FLAG_BOTTOM_UP_ONLY).bfs(roots)
    torch.cuda.synchronize()
    adj = oracle.Adjacency(n, src, dst)
    ref = np.stack([adj.bfs(s) for s in roots])
    assert (r.level.cpu().numpy() == ref).all()
    rows = {}
    for a, b in zip(src.tolist(), dst.tolist()):
        rows.setdefault(a, []).append(b)
        rows.setdefault(b, []).append(a)
    rows = {v: sorted(x, reverse=True) for v, x in rows.items()}
    for k in range(r.n_levels):
        fm, vis, active = {}, {}, 0
        for b in range(len(roots)):
            for v in np.flatnonzero(ref[b] == k).tolist():
                fm[v] = fm.get(v, 0) | 1 << b
                active |= 1 << b
            for v in np.flatnonzero((ref[b] >= 0) & (ref[b] <= k)).tolist():
                vis[v] = vis.get(v, 0) | 1 << b
        fm = {v: fm.get(v, 0) for v in rows}
        want = sum(_read(x, fm, active & ~vis.get(v, 0)) for v, x in rows.items() if active & ~vis.get(v, 0))
        assert r.stats[k]["edges"] == want, k

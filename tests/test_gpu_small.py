"""One-launch searches of small graphs against the level-by-level kernels
(which per-kernel timing selects) and the oracle: sizes around the rule's
limits, every processor count class, both directions, with and without the
sieve, long rows, and levels past the kept ones."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import require_gpu, u64

pytestmark = pytest.mark.gpu
KEYS = ("frontier", "edges", "view_bits", "sieved_bits", "unsieved_bits", "raw_bytes", "wah_unsieved_bytes",
        "wah_sieved_bytes", "self_bytes", "max_rank_bytes", "pulled", "direction", "push")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _graph(kind, n, m, seed):
    rng = np.random.default_rng(seed)
    if kind == "er":
        src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    elif kind == "hubs":  # rows far above the length a wave pushes by itself, and more of them than the queue holds
        src, dst = rng.integers(0, min(n, 700), m), rng.integers(0, n, m)
    else:  # path: one vertex a level
        src, dst = np.arange(n - 1), np.arange(1, n)
    return src.astype(np.int64), dst.astype(np.int64)


def _check(src, dst, n, p, flags, roots, max_levels=64, streams=True):
    from paper_1208_5542_amd import csbfs
    g = csbfs.Graph(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), n, p)
    adj = oracle.Adjacency(n, src, dst)
    one = csbfs.Engine(g, max_levels=max_levels, flags=flags | csbfs.FLAG_KEEP_STREAMS)
    ref = csbfs.Engine(g, max_levels=max_levels, flags=flags | csbfs.FLAG_KEEP_STREAMS | csbfs.FLAG_TIMING)
    for root in roots:
        a, b = one.bfs(root), ref.bfs(root)
        torch.cuda.synchronize()
        lev = adj.bfs(root)
        assert (a.level.cpu().numpy() == lev).all()
        assert torch.equal(a.parent, b.parent) and a.n_levels == b.n_levels == lev.max() + 1
        assert [[s[k] for k in KEYS] for s in a.stats] == [[s[k] for k in KEYS] for s in b.stats]
        kept = min(a.n_levels, max_levels)
        assert (one.stream_words(kept) == ref.stream_words(kept)).all()
        for k in range(1, kept if streams else 0):
            for i in range(p):
                for j in range(p):
                    assert u64(one.stream(k, i, j)).tolist() == u64(ref.stream(k, i, j)).tolist(), (k, i, j)


@pytest.mark.parametrize("kind,n,m,p", [
    ("er", 64, 100, 1), ("er", 128, 3, 2), ("er", 64 * 63, 9000, 1), ("er", 64 * 64, 30000, 4),
    ("er", 64 * 7 * 9, 20000, 7), ("er", 64 * 64, 40000, 64), ("er", 1 << 14, 1 << 17, 8),
    ("er", (1 << 15) - 64, 1 << 17, 1), ("er", 1 << 15, 1 << 17, 1), ("er", (1 << 15) + 64, 1 << 17, 1),
    ("hubs", 1 << 13, 1 << 18, 2), ("hubs", 1 << 13, 3 << 17, 1), ("hubs", 1 << 13, (3 << 17) + 1, 1)])
@pytest.mark.parametrize("mode", ["auto", "top_down", "bottom_up", "no_sieve"])
def test_one_launch_search(kind, n, m, p, mode):
    from paper_1208_5542_amd import csbfs
    flags = {"auto": 0, "top_down": csbfs.FLAG_SPARSE_ONLY, "bottom_up": csbfs.FLAG_BOTTOM_UP_ONLY,
             "no_sieve": csbfs.FLAG_NO_SIEVE}[mode]
    src, dst = _graph(kind, n, m, n + p)
    _check(src, dst, n, p, flags, [int(src[0]), int(dst[1]), n - 1], streams=p < 64)


@pytest.mark.parametrize("max_levels", [1, 2, 17, 300])
def test_levels_past_the_kept_ones(max_levels):
    src, dst = _graph("path", 192, 0, 0)
    _check(src, dst, 192, 3, 0, [0, 191, 96], max_levels=max_levels)


def test_caller_memory_without_mailbox():
    from paper_1208_5542_amd import csbfs
    n, p = 1 << 12, 4
    src, dst = _graph("er", n, 1 << 15, 5)
    g = csbfs.Graph(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), n, p)
    adj = oracle.Adjacency(n, src, dst)
    cfg = csbfs.search_config(max_levels=64)
    eng = csbfs.WorkspaceSearch(g, cfg)
    level = torch.empty(n, dtype=torch.int32, device="cuda")
    parent = torch.empty(n, dtype=torch.int32, device="cuda")
    import ctypes
    nl = ctypes.c_int32()
    ws = torch.full((csbfs.layout_query(n, src.size, p, cfg)["workspace_bytes"],), 255, dtype=torch.uint8,
                    device="cuda")
    for root in (int(src[0]), 7):
        rc = csbfs.lib().csbfs_bfs_ws(g.handle, root, ctypes.byref(cfg), level.data_ptr(), parent.data_ptr(), None, 0,
                                      ctypes.byref(nl), ws.data_ptr(), ws.numel(), None,
                                      torch.cuda.current_stream().cuda_stream)
        assert rc == csbfs.OK and nl.value == adj.bfs(root).max() + 1
        assert (level.cpu().numpy() == adj.bfs(root)).all()
        r = eng.bfs(root)
        assert torch.equal(r.level, level) and torch.equal(r.parent, parent)


@pytest.mark.parametrize("n,p", [(1 << 22, 2), ((1 << 22) + 128, 2)])
def test_sizes_around_the_eager_kernels(n, p):
    """The level kernels that load at once and those that follow block marks:
    same levels as the oracle, same parents and messages in either direction."""
    from paper_1208_5542_amd import csbfs
    rng = np.random.default_rng(n)
    used = rng.choice(n, 40000, replace=False)  # most blocks of 4096 vertices stay empty
    used = used[(used // 4096) % 3 == 0]
    src, dst = used[rng.integers(0, used.size, 200000)], used[rng.integers(0, used.size, 200000)]
    g = csbfs.Graph(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), n, p)
    ref = oracle.Adjacency(n, src, dst).bfs(int(src[0]))
    rows = []
    for flags in (0, csbfs.FLAG_SPARSE_ONLY, csbfs.FLAG_BOTTOM_UP_ONLY):
        eng = csbfs.Engine(g, flags=flags)
        r = eng.bfs(int(src[0]))
        assert (r.level.cpu().numpy() == ref).all(), flags
        rows.append((r.parent, eng.stream_words(r.n_levels), [s["view_bits"] for s in r.stats]))
    for parent, words, bits in rows[1:]:
        assert torch.equal(parent, rows[0][0]) and (words == rows[0][1]).all() and bits == rows[0][2]

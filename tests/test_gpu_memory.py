"""Caller-owned memory (the problem statement of Sec. II: the caller holds
the graph and the search state): graphs built into caller buffers, searches
in caller workspaces with and without a pinned mailbox, exact buffer sizes,
and the block-row sort on rows of every length class. Every result is
checked against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1208_5542_amd import inputs
from tests.gpu_util import from_words, log, require_gpu, u64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int64)).cuda()


def _check(csbfs, eng, n, p, src, dst, root, adj, V, keep=True):
    r = eng.bfs(root)
    torch.cuda.synchronize()
    lev = r.level.cpu().numpy()
    par = r.parent.cpu().numpy()
    ref = adj.alg3(p, V, root, dump=keep)
    assert (lev == ref.level).all(), "level"
    assert (par == ref.parent).all(), "parent"
    assert r.n_levels == ref.n_levels
    assert (eng.stream_words(r.n_levels) == ref.words).all()
    if keep:
        for k in range(1, r.n_levels):
            for i in range(p):
                for j in range(p):
                    got = u64(eng.stream(k, i, j))
                    assert got.tolist() == ref.streams[k, i, j, : ref.words[k, i, j]].tolist(), (k, i, j)
    lb = ref.level_bytes()
    for k in range(r.n_levels):
        assert r.stats[k]["wah_sieved_bytes"] == lb[k]["wah_sieved"]
        assert r.stats[k]["max_rank_bytes"] == lb[k]["max_rank_volume"]
    return r


@pytest.mark.parametrize("scale,p", [(10, 1), (11, 4), (12, 8), (13, 2)])
def test_caller_graph_equals_library_graph(scale, p):
    from paper_1208_5542_amd import csbfs
    src, dst = inputs.rmat_tuples(scale, 16)
    n = 1 << scale
    a = csbfs.Graph(_dev(src), _dev(dst), n, p)
    b = csbfs.Graph(_dev(src), _dev(dst), n, p, memory="caller")
    assert b.memory.numel() == csbfs.layout_query(n, len(src), p)["graph_bytes"]
    assert a.info.nnz == b.info.nnz == 2 * len(src)
    assert torch.equal(a.directory(), b.directory())
    for i in range(p):
        for j in range(p):
            ra, ca = a.block(i, j)
            rb, cb = b.block(i, j)
            assert torch.equal(ra, rb) and torch.equal(ca, cb), (i, j)


@pytest.mark.parametrize("mode", [0, 8, 16, 32])
@pytest.mark.parametrize("mailbox", [True, False])
def test_workspace_search_matches_oracle(mode, mailbox):
    from paper_1208_5542_amd import csbfs
    scale, p = 12, 4
    src, dst = inputs.rmat_tuples(scale, 16)
    n = 1 << scale
    g = csbfs.Graph(_dev(src), _dev(dst), n, p, memory="caller")
    cfg = csbfs.search_config(flags=csbfs.FLAG_KEEP_STREAMS | mode, max_levels=32)
    eng = csbfs.WorkspaceSearch(g, cfg, mailbox=mailbox)
    eng.workspace.fill_(0xA5)  # any contents: the search clears what it needs
    adj = oracle.Adjacency(n, src, dst)
    V = oracle.directory(n, p, src, dst).reshape(-1)
    for root in inputs.pick_roots(n, src, dst, 3, inputs.graph_seed(scale) + 2):
        log(f"workspace search mode={mode} mailbox={mailbox} root={int(root)}")
        _check(csbfs, eng, n, p, src, dst, int(root), adj, V)


def test_workspace_and_engine_agree_at_scale_20():
    from paper_1208_5542_amd import csbfs
    scale, p = 20, 4
    src, dst = inputs.rmat_tuples(scale, 16)
    n = 1 << scale
    g = csbfs.Graph(_dev(src), _dev(dst), n, p, memory="caller")
    ws = csbfs.WorkspaceSearch(g, csbfs.search_config(max_levels=64))
    eng = csbfs.Engine(g, max_levels=64)
    adj = oracle.Adjacency(n, src, dst)
    for root in inputs.pick_roots(n, src, dst, 3, inputs.graph_seed(scale) + 2):
        a = ws.bfs(int(root))
        la, pa = a.level.clone(), a.parent.clone()
        b = eng.bfs(int(root))
        assert torch.equal(la, b.level) and torch.equal(pa, b.parent)
        assert a.n_levels == b.n_levels
        assert [s["wah_sieved_bytes"] for s in a.stats] == [s["wah_sieved_bytes"] for s in b.stats]
        ref = adj.bfs(int(root))
        assert (la.cpu().numpy() == ref).all()
        assert (pa.cpu().numpy() == adj.parents_max(ref, int(root))).all()


def test_exact_sizes_and_argument_checks():
    from paper_1208_5542_amd import csbfs
    L = csbfs.lib()
    scale, p = 11, 4
    src, dst = inputs.rmat_tuples(scale, 16)
    n, m = 1 << scale, len(src)
    sz = csbfs.layout_query(n, m, p)
    s, d = _dev(src), _dev(dst)
    gm = torch.empty(sz["graph_bytes"], dtype=torch.uint8, device="cuda")
    sm = torch.empty(sz["build_scratch_bytes"], dtype=torch.uint8, device="cuda")
    h = ctypes.c_void_p()
    ptr = lambda t, off=0: ctypes.c_void_p(t.data_ptr() + off)
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.csbfs_graph_build_into(ptr(s), ptr(d), m, n, p, ptr(gm), gm.numel() - 1, ptr(sm), sm.numel(),
                                    st, ctypes.byref(h)) == csbfs.ENOSPACE
    assert L.csbfs_graph_build_into(ptr(s), ptr(d), m, n, p, ptr(gm), gm.numel(), ptr(sm), sm.numel() - 1,
                                    st, ctypes.byref(h)) == csbfs.ENOSPACE
    assert L.csbfs_graph_build_into(ptr(s), ptr(d), m, n, p, ptr(gm, 8), gm.numel() - 8, ptr(sm),
                                    sm.numel(), st, ctypes.byref(h)) == csbfs.EINVAL
    assert L.csbfs_graph_build_into(ptr(s), ptr(d), m, n, p, ptr(gm), gm.numel(), ptr(sm), sm.numel(),
                                    st, ctypes.byref(h)) == csbfs.OK
    del sm
    cfg = csbfs.search_config()
    ws = torch.empty(sz["workspace_bytes"], dtype=torch.uint8, device="cuda")
    lev = torch.empty(n, dtype=torch.int32, device="cuda")
    par = torch.empty(n, dtype=torch.int32, device="cuda")
    nl = ctypes.c_int32()
    root = int(inputs.pick_roots(n, src, dst, 1, 7)[0])
    args = (h, root, ctypes.byref(cfg), ptr(lev), ptr(par), None, 0, ctypes.byref(nl))
    assert L.csbfs_bfs_ws(*args, ptr(ws), ws.numel() - 1, None, st) == csbfs.ENOSPACE
    assert L.csbfs_bfs_ws(*args, ptr(ws, 64), ws.numel() - 64, None, st) == csbfs.EINVAL
    bad = torch.zeros(2, dtype=torch.int64)  # pageable, not pinned
    assert L.csbfs_bfs_ws(*args, ptr(ws), ws.numel(), ctypes.c_void_p(bad.data_ptr()), st) == csbfs.EINVAL
    assert L.csbfs_bfs_ws(h, n, ctypes.byref(cfg), ptr(lev), ptr(par), None, 0, ctypes.byref(nl), ptr(ws),
                          ws.numel(), None, st) == csbfs.ERANGE
    bad_cfg = csbfs.search_config(flags=csbfs.FLAG_TIMING)
    assert L.csbfs_bfs_ws(h, root, ctypes.byref(bad_cfg), ptr(lev), ptr(par), None, 0, ctypes.byref(nl),
                          ptr(ws), ws.numel(), None, st) == csbfs.EINVAL
    rc = L.csbfs_bfs_ws(*args, ptr(ws), ws.numel(), None, st)
    assert rc == csbfs.OK, L.csbfs_last_error().decode()
    adj = oracle.Adjacency(n, src, dst)
    assert (lev.cpu().numpy() == adj.bfs(root)).all()
    assert L.csbfs_graph_free(h) == 0


def test_row_sort_every_length_class():
    """Block rows of every length class of the build's row sort (thread, wave,
    workgroup network, radix) come out in decreasing order with the right
    entries, and the search on that graph equals the oracle."""
    from paper_1208_5542_amd import csbfs
    rng = np.random.default_rng(11)
    n, p = 1 << 16, 2
    R = n // p
    parts = []
    # hubs: rows of about 40000, 5000, 600, 20 entries (duplicates included)
    for hub, deg in ((3, 40000), (70001 % n, 5000), (12345, 600), (54321, 20)):
        parts.append((np.full(deg, hub), rng.integers(0, n, deg)))
    parts.append((rng.integers(0, n, 60000), rng.integers(0, n, 60000)))
    src = np.concatenate([a for a, _ in parts]).astype(np.int64)
    dst = np.concatenate([b for _, b in parts]).astype(np.int64)
    for memory in ("library", "caller"):
        g = csbfs.Graph(_dev(src), _dev(dst), n, p, memory=memory)
        a = np.r_[src, dst]
        b = np.r_[dst, src]
        lens = []
        for i in range(p):
            for j in range(p):
                rp, col = g.block(i, j)
                rp, col = rp.cpu().numpy(), col.cpu().numpy().astype(np.int64)
                sel = (a // R == j) & (b // R == i)
                order = np.lexsort((-(b[sel] - i * R), a[sel] - j * R))
                exp_col = (b[sel] - i * R)[order]
                exp_rp = np.r_[0, np.cumsum(np.bincount(a[sel] - j * R, minlength=R))]
                assert (rp == exp_rp).all(), (i, j)
                assert (col == exp_col).all(), (i, j)
                lens.append(int(np.diff(rp).max()))
        assert max(lens) > 16384
        adj = oracle.Adjacency(n, src, dst)
        V = oracle.directory(n, p, src, dst).reshape(-1)
        eng = csbfs.Engine(g, max_levels=64)
        for root in (3, 12345, int(src[-1])):
            r = eng.bfs(root)
            ref = adj.alg3(p, V, root)
            assert (r.level.cpu().numpy() == ref.level).all()
            assert (r.parent.cpu().numpy() == ref.parent).all()


@pytest.mark.parametrize("mailbox", [True, False])
@pytest.mark.parametrize("max_levels", [1, 2, 63, 64])
def test_level_count_past_the_kept_levels(max_levels, mailbox):
    """Levels that share the last record are counted all the same, also where
    the host reads each level's size from that record."""
    from paper_1208_5542_amd import csbfs
    n, p = 64 * 600, 3
    src = np.arange(64, dtype=np.int64)
    g = csbfs.Graph(_dev(src), _dev(src + 1), n, p)
    cfg = csbfs.search_config(max_levels=max_levels, segment_groups=1024)  # the level-by-level kernels
    eng = csbfs.WorkspaceSearch(g, cfg, mailbox=mailbox)
    for root, levels in ((0, 65), (40, 41), (100, 1)):
        r = eng.bfs(root)
        assert r.n_levels == levels == int(r.level.max()) + 1
        assert [s["frontier"] for s in r.stats[1:]] == [1 + (root > 0 and k <= 24) for k in range(1, min(levels, max_levels))]

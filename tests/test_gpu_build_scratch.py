"""Builds that cannot have the sort's scratch count instead: the same graph in
the scratch that the header says is enough, and a refusal below it."""
import ctypes

import numpy as np
import pytest
import torch

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _build(src, dst, n, p, scratch_bytes):
    """(status, (row_ptr, col) of every block, directory, searches that use the rest of the graph)."""
    from paper_1208_5542_amd import csbfs
    L = csbfs.lib()
    gb = csbfs.layout_query(n, src.numel(), p)["graph_bytes"]
    gm = torch.full((gb,), 0x5A, dtype=torch.uint8, device="cuda")
    sm = torch.full((scratch_bytes,), 0xA5, dtype=torch.uint8, device="cuda")
    h = ctypes.c_void_p()
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    rc = L.csbfs_graph_build_into(ptr(src), ptr(dst), src.numel(), n, p, ptr(gm), gb, ptr(sm), scratch_bytes,
                                  ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), ctypes.byref(h))
    if rc != csbfs.OK:
        return rc, None
    # a handle like the binding's own
    g = csbfs.Graph.__new__(csbfs.Graph)
    g._h, g.memory, g.n_tuples, g.n, g.p, g.range = h, gm, src.numel(), n, p, n // p
    out = [g.block(i, j) for i in range(p) for j in range(p)] + [g.directory()]
    for flags in (csbfs.FLAG_SPARSE_ONLY, csbfs.FLAG_BOTTOM_UP_ONLY):
        r = csbfs.Engine(g, flags=flags).bfs(int(src[0]))
        out += [r.level, r.parent, r.stats]
    g.close()
    return rc, out


def _same(a, b):
    if isinstance(a, torch.Tensor):
        return torch.equal(a, b)
    if isinstance(a, (tuple, list)) and not isinstance(a[0], dict):
        return len(a) == len(b) and all(_same(x, y) for x, y in zip(a, b))
    return a == b


# entry counts around the sort's rule, sizes whose rows end within a wave or
# span many, ranges that are no power of two, and one row that holds everything
@pytest.mark.parametrize("m,n,p,top", [(1 << 17, 64, 1, 64), (1 << 17, 64 * 64, 64, 64 * 64), (1 << 17, 3 * 64 * 683, 3, 1 << 17),
                                       (200003, 1 << 16, 4, 1 << 16), (200003, 1 << 16, 1, 3), (1 << 19, 7 * 64 * 50, 7, 900),
                                       (131073, 1 << 20, 2, 1 << 20)])
def test_the_same_graph_in_less_scratch(m, n, p, top):
    from paper_1208_5542_amd import csbfs
    g = torch.Generator(device="cuda").manual_seed(m + n)
    src = torch.randint(0, min(top, n), (m,), generator=g, device="cuda")
    dst = torch.randint(0, n, (m,), generator=g, device="cuda")
    need = csbfs.layout_query(n, m, p)["build_scratch_bytes"]
    less = 4 * p * n + p * n // 64 + 5 * m // 8 + 16 * p * p + 8192
    rc, full = _build(src, dst, n, p, need)
    assert rc == csbfs.OK
    rc, counted = _build(src, dst, n, p, min(less, need - 1))
    assert rc == (csbfs.OK if less < need else csbfs.ENOSPACE)
    assert less >= need or _same(full, counted)
    assert _build(src, dst, n, p, min(4 * p * n, 8 * 2 * m) - 1)[0] == csbfs.ENOSPACE
    a, b = src.cpu().numpy(), dst.cpu().numpy()
    a, b = np.r_[a, b], np.r_[b, a]
    R = n // p
    for q in range(p * p):
        rp, col = (x.cpu().numpy() for x in full[q])
        sel = (b // R == q // p) & (a // R == q % p)
        u, v = a[sel] - (q % p) * R, b[sel] - (q // p) * R
        assert (rp == np.r_[0, np.cumsum(np.bincount(u, minlength=R))]).all(), q
        assert (col.astype(np.int64) == v[np.lexsort((-v, u))]).all(), q


def test_build_with_no_room_for_the_sort():
    """csbfs_graph_build on a card with room for the graph and the counting
    build's scratch, and not for the 4.1 GiB that sorting 2^29 entries takes."""
    from paper_1208_5542_amd import csbfs
    n, m, p = 1 << 20, 1 << 28, 4
    src = torch.randint(0, n, (m,), device="cuda")
    dst = torch.randint(0, n, (m,), device="cuda")
    torch.cuda.empty_cache()
    left = csbfs.layout_query(n, m, p)["graph_bytes"] + (800 << 20)  # blocks the library keeps: 2 GiB at most
    free = torch.cuda.mem_get_info()[0]
    if free < left:
        pytest.skip("needs 6 GiB of device memory")
    held = torch.empty(free - left, dtype=torch.uint8, device="cuda")
    g = csbfs.Graph(src, dst, n, p)
    del held
    torch.cuda.empty_cache()
    assert g.info.nnz == 2 * m
    R = n // p
    rp, col = g.block(1, 2)  # sources in R_2, targets in R_1
    a, b = torch.cat([src, dst]), torch.cat([dst, src])
    sel = (a // R == 2) & (b // R == 1)
    key = (a[sel] - 2 * R) * R + (R - 1 - (b[sel] - R))
    key, _ = key.sort()
    assert torch.equal(col.long(), R - 1 - key % R)
    assert torch.equal(rp[1:].long(), torch.bincount(key // R, minlength=R).cumsum(0))
    g.close()

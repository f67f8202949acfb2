"""A row of almost 2^31 entries, the longest a block may hold: positions in it
plus one step of a kernel's loop pass 2^31. The graph is one vertex with
2^30 - 10 self-loops and nine edges, so every result is known."""
import pytest
import torch

from tests.gpu_util import log, require_gpu

pytestmark = pytest.mark.gpu
N, M, H = 64 * 64, (1 << 30) - 1, 1000
ABOVE, BELOW = [4095, 3000, 2999, 2048, 1500, 1100, 1064, 1001], 17


@pytest.fixture(scope="module")
def graph():
    require_gpu()
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GiB of device memory")
    from paper_1208_5542_amd import csbfs
    src = torch.full((M,), H, dtype=torch.int64, device="cuda")
    dst = src.clone()
    dst[:8] = torch.tensor(ABOVE, device="cuda")
    src[M - 1] = BELOW
    log(f"build of {M} tuples")
    g = csbfs.Graph(src, dst, N, 1)
    del src, dst
    torch.cuda.empty_cache()
    yield g
    g.close()


def _loops():
    return 2 * (M - 9)


def test_block_of_the_longest_row(graph):
    row = _loops() + 9
    assert graph.info.max_block_nnz == graph.info.nnz == 2 * M == (1 << 31) - 2
    rp, col = graph.block(0, 0)
    assert int(rp[H]) == 1 and int(rp[H + 1]) - 1 == row and int(rp[N]) == 2 * M
    got = col[1:1 + row]
    assert got[:8].tolist() == ABOVE and int(got[-1]) == BELOW
    lo, hi = torch.aminmax(got[8:-1])
    assert int(lo) == int(hi) == H


def test_searches_over_the_longest_row(graph):
    from paper_1208_5542_amd import csbfs
    level = torch.full((N,), -1, dtype=torch.int32, device="cuda")
    level[ABOVE + [BELOW]] = 2
    level[H], level[ABOVE[0]] = 1, 0
    for flags in (csbfs.FLAG_SPARSE_ONLY, 0):
        log(f"search flags={flags}")
        r = csbfs.Engine(graph, flags=flags).bfs(ABOVE[0])
        assert torch.equal(r.level, level) and r.parent[ABOVE[1:] + [BELOW]].unique().tolist() == [H]
        if flags:
            assert r.stats[1]["edges"] == _loops() + 9
        log(f"batch flags={flags}")
        b = csbfs.BatchEngine(graph, max_roots=2, flags=flags).bfs([ABOVE[0], H])
        assert torch.equal(b.level[0], level)
        assert int(b.level[1, H]) == 0 and b.level[1, ABOVE + [BELOW]].unique().tolist() == [1]
        if flags:
            assert b.stats[1]["edges"] == _loops() + 9 + 9


def test_bottom_up_finds_the_rows_last_entry(graph):
    """The frontier neighbour is the last entry of the row, so a workgroup
    reads all of it, and the merged row's end is seen to be in place."""
    from paper_1208_5542_amd import csbfs
    log("batch bottom-up")
    b = csbfs.BatchEngine(graph, max_roots=1, flags=csbfs.FLAG_BOTTOM_UP_ONLY).bfs([BELOW])
    assert int(b.level[0, H]) == 1 and b.level[0, ABOVE].unique().tolist() == [2]
    assert b.stats[0]["edges"] >= _loops() + 9

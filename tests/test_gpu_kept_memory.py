"""Device memory that the library keeps of freed graphs: given back on request,
and counted in full by the graph that takes it over."""
import pytest
import torch

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu
MIB = 1 << 20


@pytest.fixture(autouse=True)
def _fresh():
    require_gpu()
    from paper_1208_5542_amd import csbfs
    csbfs.trim()
    yield
    csbfs.trim()


def _tuples(n, m):
    return torch.randint(0, n, (m,), device="cuda"), torch.randint(0, n, (m,), device="cuda")


def test_trim_gives_kept_blocks_back():
    from paper_1208_5542_amd import csbfs
    src, dst = _tuples(1 << 20, 1 << 24)
    sz = csbfs.layout_query(1 << 20, 1 << 24, 4)
    g = csbfs.Graph(src, dst, 1 << 20, 4)
    live = csbfs.Graph(src[:MIB].contiguous(), dst[:MIB].contiguous(), 1 << 20, 4)
    ref = live.block(2, 3)
    g.close()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    csbfs.trim()
    # the freed graph and the scratch of its build, at least
    assert torch.cuda.mem_get_info()[0] - before >= sz["graph_bytes"] + sz["build_scratch_bytes"]
    assert all(torch.equal(a, b) for a, b in zip(ref, live.block(2, 3)))
    live.close()
    csbfs.trim()
    csbfs.trim()  # nothing kept
    g = csbfs.Graph(src, dst, 1 << 20, 4)
    assert g.info.nnz == 1 << 25


def test_device_bytes_of_a_graph_in_a_reused_block():
    from paper_1208_5542_amd import csbfs
    n, m = 1 << 20, 1 << 23
    src, dst = _tuples(n, m)
    a = csbfs.Graph(src, dst, n, 2)
    assert a.info.device_bytes == csbfs.layout_query(n, m, 2)["graph_bytes"]
    a.close()
    less = m - m // 10
    free = torch.cuda.mem_get_info()[0]
    b = csbfs.Graph(src[:less], dst[:less], n, 2)
    assert torch.cuda.mem_get_info()[0] == free  # both blocks were kept ones
    assert b.info.device_bytes == a.info.device_bytes > csbfs.layout_query(n, less, 2)["graph_bytes"]
    c = csbfs.Graph(src[:less], dst[:less], n, 2, memory="caller")
    assert c.info.device_bytes == csbfs.layout_query(n, less, 2)["graph_bytes"]

"""The row sort of builds that count (csrc/csbfs/sort.hip), at the lengths of its
radix class: rows above 16384 entries, around its chunks of 8192, with an even and
an odd number of 4-bit passes (the last pass ends in the row or in the temp
buffer). Small builds count by themselves, larger ones in a scratch that only
covers counting; both against numpy, and against the build that sorts."""
import numpy as np
import pytest
import torch

from tests.gpu_util import require_gpu
from tests.test_gpu_build_scratch import _build, _same

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _counting(n, m, p):
    return 4 * p * n + p * n // 64 + 5 * m // 8 + 16 * p * p + 8192


# |R| of 64, 192, 1024, 10944 and 2^17 vertices: 2, 2, 3, 4 and 5 passes
@pytest.mark.parametrize("R", [64, 192, 1024, 64 * 171, 1 << 17])
@pytest.mark.parametrize("p", [1, 3])
@pytest.mark.parametrize("length", [16384, 16385, 24576, 24577, 50000, 100003, 300000])
def test_long_rows(length, p, R):
    from paper_1208_5542_amd import csbfs
    n = p * R
    rng = np.random.default_rng(length + R + p)
    hub, lo = n - 7, R * int(rng.integers(0, p))
    few = 5000
    # the hub's row of one block has `length` entries: few of them come from the other tuples' side
    src = np.r_[np.full(length, hub), rng.integers(0, n, few)]
    dst = np.r_[lo + rng.integers(0, R, length), rng.integers(0, n, few)]
    m = src.size
    s, d = (torch.from_numpy(x.astype(np.int64)).cuda() for x in (src, dst))
    need = csbfs.layout_query(n, m, p)["build_scratch_bytes"]
    small = 2 * m < 1 << 18
    scratch = need if small else min(need - 1, _counting(n, m, p))
    if not small and _counting(n, m, p) >= need:
        pytest.skip("the sort's scratch is the smaller one")
    rc, got = _build(s, d, n, p, scratch)
    assert rc == csbfs.OK
    a, b = np.r_[src, dst], np.r_[dst, src]
    longest = 0
    for q in range(p * p):
        rp, col = (x.cpu().numpy() for x in got[q])
        sel = (b // R == q // p) & (a // R == q % p)
        u, v = a[sel] - (q % p) * R, b[sel] - (q // p) * R
        assert (rp == np.r_[0, np.cumsum(np.bincount(u, minlength=R))]).all(), q
        assert (col.astype(np.int64) == v[np.lexsort((-v, u))]).all(), q
        longest = max(longest, int(np.diff(rp).max()))
    assert longest >= length
    if not small:
        assert _same(got, _build(s, d, n, p, need)[1])

"""One-launch searches at the limits of their rule: state that fills the LDS, as
many streams as they are made with, and as many entries, each beside the next
size, which goes to the level-by-level kernels."""
import pytest

from tests.gpu_util import require_gpu
from tests.test_gpu_small import _check, _graph

pytestmark = pytest.mark.gpu

# (vertices, processors, tuples, made in one launch?); 3 << 17 tuples have as
# many entries as the rule admits
LIMITS = [(32512, 1, 3 << 17, True), (32512, 1, (3 << 17) + 1, False), (32576, 1, 60000, False),
          (30080, 2, 90000, True), (30208, 2, 90000, False), (26112, 4, 60000, True), (26368, 4, 60000, False),
          (26560, 5, 60000, True), (26880, 5, 60000, False), (22528, 8, 50000, True), (23040, 8, 50000, False),
          (13376, 11, 30000, True), (14080, 11, 30000, False), (4992, 13, 9000, True), (5824, 13, 9000, False),
          (896, 14, 4000, True), (1792, 14, 4000, False), (1024, 16, 4000, False), (4096, 64, 40000, False)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("n,p,m,one", LIMITS)
def test_searches_at_the_limits(n, p, m, one):
    from paper_1208_5542_amd import csbfs
    src, dst = _graph("er", n, m, n + p)
    roots = [int(src[0]), n - 1]
    for flags in (0, csbfs.FLAG_SPARSE_ONLY, csbfs.FLAG_BOTTOM_UP_ONLY):
        _check(src, dst, n, p, flags, roots, streams=flags == 0 and p < 16)

"""Decoding at the edge of what a chunk lays out in LDS: two groups a word and 64
(streams of up to 2^19 words in chunks of 1024 words, longer ones of 2048)."""
import numpy as np
import pytest
import torch

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("ones", [0, 1])
@pytest.mark.parametrize("extra", [-1, 0, 62, 63, 64, 65, 66, 500])
@pytest.mark.parametrize("words,chunk", [(3 * 1024, 1024), (2047, 1024), ((1 << 19) + 6 * 1024 + 7, 2048)])
def test_chunks_of_two_groups_a_word(words, chunk, extra, ones):
    from paper_1208_5542_amd import csbfs
    # literals (the first bit of their group) and fills of three groups in turn;
    # the first fill of every other chunk is `extra` groups longer
    w = np.full(words, 1 << 62, dtype=np.uint64)
    count = np.ones(words, dtype=np.int64)
    fill = np.arange(1, words, 2)
    count[fill] = 3
    count[fill[fill % (2 * chunk) == 1]] = 3 + extra
    w[fill] = (2 + ones << 62) + count[fill].astype(np.uint64)
    first = np.r_[0, np.cumsum(count)]
    nbits = int(first[-1]) * 63
    bits = np.zeros((nbits + 63) // 64 * 64, dtype=np.uint8)
    bits[first[:-1:2] * 63] = 1
    if ones:
        edge = np.zeros(first[-1] + 1, dtype=np.int8)
        edge[first[fill]] += 1
        edge[first[fill + 1]] -= 1
        bits[:nbits].reshape(-1, 63)[np.cumsum(edge[:-1]) > 0] = 1
    out, status = csbfs.wah_decode_or(torch.from_numpy(w.view(np.int64)).cuda(), nbits)
    assert status == 0
    assert (out.cpu().numpy() == np.packbits(bits, bitorder="little").view(np.int64)).all()

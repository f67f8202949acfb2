"""Decoding streams from elsewhere at the edges of its chunks (1024 words, and
2048 above 2^19 words): stream lengths around their multiples, fills that span
chunks, words past the chunk's staged groups, and streams that are wrong in a
late chunk."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import from_words, require_gpu, to_words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _decode(words, nbits, dst=None):
    from paper_1208_5542_amd import csbfs
    return csbfs.wah_decode_or(torch.from_numpy(np.ascontiguousarray(words).view(np.int64)).cuda(), nbits, dst=dst)


@pytest.mark.parametrize("groups", [1023, 1024, 1025, 2048, 2049, 40 * 1024, (1 << 19) - 1, 1 << 19, (1 << 19) + 1,
                                    (1 << 19) + 2048, (1 << 19) + 4097])
@pytest.mark.parametrize("tail", [0, 17])
def test_literal_streams(groups, tail):
    # alternating bits: every group is a literal, one word each
    nbits = groups * 63 + tail
    a = (np.arange(nbits) % 3 == 0).astype(np.uint8)
    words = oracle.wah_encode(a)
    assert len(words) == groups + (tail > 0)
    b = (np.arange(nbits) % 5 == 0).astype(np.uint8)
    out, status = _decode(words, nbits, to_words(b))
    assert status == 0 and (from_words(out, nbits) == (a | b)).all()


@pytest.mark.parametrize("seed", range(4))
def test_fills_over_chunks(seed):
    rng = np.random.default_rng(seed)
    parts = []
    for _ in range(6000):
        kind = rng.integers(0, 4)
        length = int(rng.integers(1, 40)) * 63 if kind < 2 else 63 * int(rng.integers(1, 4))
        if rng.random() < 0.001:
            length *= 400  # far beyond what a chunk stages
        parts.append(np.full(length, kind, np.uint8) if kind < 2 else rng.integers(0, 2, length).astype(np.uint8))
    a = np.concatenate(parts + [rng.integers(0, 2, 31).astype(np.uint8)])
    words = oracle.wah_encode(a)
    assert len(words) > 3 * 1024
    out, status = _decode(words, a.size)
    assert status == 0 and (from_words(out, a.size) == a).all()


def test_wrong_late_chunks():
    Z = 1 << 63
    nbits = 63 * 5000 + 11
    good = np.full(5001, 5, dtype=np.uint64)
    good[-1] = 1
    assert _decode(good, nbits)[1] == 0
    for at, word in ((3000, Z), (4500, Z | 2), (2048, Z | (1 << 61)), (4999, Z | 9), (5000, 1 << 11)):
        bad = good.copy()
        bad[at] = word
        assert _decode(bad, nbits)[1] != 0, (at, word)
    assert _decode(np.delete(good, 1500), nbits)[1] != 0

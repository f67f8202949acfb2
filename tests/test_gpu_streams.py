"""Codec calls of the binding on a stream other than torch's current one: the
call's scratch and status tensors belong to the current stream, so its result
must not be read, nor its scratch reused, before the other stream is done."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import from_words, require_gpu, to_words, u64

pytestmark = pytest.mark.gpu
NBITS = 63 * 3000 + 17


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _busy_stream():
    """A stream with some milliseconds of work queued, so that what follows on
    it is still waiting when a call that does not wait returns."""
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        torch.cuda._sleep(20_000_000)
    return s


def _bits():
    return (np.random.default_rng(5).random(NBITS) < 0.02).astype(np.uint8)


def test_decode_status_and_result_on_another_stream():
    from paper_1208_5542_amd import csbfs
    bits = _bits()
    words = csbfs.wah_encode(to_words(bits), NBITS)
    bad = words.clone()
    bad[3] = -(1 << 63)  # a fill of no groups
    torch.cuda.synchronize()
    dst, status = csbfs.wah_decode_or(words, NBITS, stream=_busy_stream())
    assert status == 0 and (from_words(dst, NBITS) == bits).all()
    _, status = csbfs.wah_decode_or(bad, NBITS, stream=_busy_stream())
    assert status != 0


def test_encode_length_on_another_stream():
    from paper_1208_5542_amd import csbfs
    bits = _bits()
    dev = to_words(bits)
    torch.cuda.synchronize()
    words = csbfs.wah_encode(dev, NBITS, stream=_busy_stream())
    assert u64(words).tolist() == oracle.wah_encode(bits).tolist()

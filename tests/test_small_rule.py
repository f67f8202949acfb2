"""The rule that sends a search to the one-launch kernel (csrc/csbfs/small_rule.hpp),
compiled by the host compiler."""
import os
import shutil
import subprocess

import pytest

from tests.test_gpu_small_limits import LIMITS

REPO = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(REPO, "tests", "sanitize")
CSRC = os.path.join(REPO, "paper_1208_5542_amd", "csrc", "csbfs")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ is not installed")
    exe = str(tmp_path_factory.mktemp("rule") / "small_rule_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(HERE, "hip_stub"), "-I", CSRC, "-I",
                    os.path.join(REPO, "include"), os.path.join(HERE, "small_rule_check.cpp"), "-o", exe], check=True)

    def ask(cases):
        text = "".join(f"{n} {p} {nnz}\n" for n, p, nnz in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return ask


def test_limits(rule):
    got = rule([(n, p, 2 * m) for n, p, m, _ in LIMITS])
    assert [bool(one) for one, _ in got] == [one for _, _, _, one in LIMITS]


def test_no_processor_count_from_15_on(rule):
    # p * p streams a level, sixteen waves: 256 of them one after another at p = 64
    cases = [(64 * p * k, p, 1000) for p in range(15, 65) for k in (1, 2, 7)]
    assert not any(one for one, _ in rule(cases))


def test_lds_of_every_admitted_size(rule):
    cases = [(n, p, 1000) for p in range(1, 15) for n in range(64 * p, (1 << 15) + 64 * p, 64 * p)]
    got = rule(cases)
    assert max(b for _, b in got) > 160 * 1024 - 2048  # the limit is reached
    assert all(b <= 160 * 1024 - 1024 for _, b in got)
    assert all(one for (n, p, _), (one, _) in zip(cases, got) if n <= 8192 and p <= 10)

"""The library's pool of device blocks on the CPU: compiled by the host compiler
with stub HIP calls (tests/sanitize/hip_stub) and run under the address,
undefined-behaviour and thread sanitizers."""
import os
import shutil
import subprocess

import pytest

REPO = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(REPO, "tests", "sanitize")
CSRC = os.path.join(REPO, "paper_1208_5542_amd", "csrc", "csbfs")


@pytest.mark.parametrize("kind", ["address,undefined", "thread"])
def test_device_block_pool(tmp_path, kind):
    if shutil.which("g++") is None:
        pytest.skip("g++ is not installed")
    exe = str(tmp_path / "pool_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-pthread", f"-fsanitize={kind}",
                    "-fno-sanitize-recover=all", "-I", os.path.join(HERE, "hip_stub"), "-I", CSRC, "-I",
                    os.path.join(REPO, "include"), os.path.join(HERE, "pool_check.cpp"), "-o", exe], check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:verify_asan_link_order=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=120)
    if "unexpected memory mapping" in r.stderr:  # a kernel whose address randomization this sanitizer does not know
        pytest.skip(r.stderr.strip())
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr

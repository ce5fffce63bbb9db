"""The pool of idle device blocks (bh_pool.h) over a scripted device, on the CPU: plain and under
the address, undefined-behaviour and thread sanitizers."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2010_08735_amd", "csrc")
SCENARIOS = ["reuse", "refused_wait", "allocation_failure", "full_pool", "larger_cycle",
             "peers", "budget", "threads"]
FLAVOURS = {"plain": ["-O2"],
            "asan_ubsan": ["-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=undefined"],
            "tsan": ["-O1", "-g", "-fsanitize=thread"]}


@pytest.fixture(scope="module", params=list(FLAVOURS))
def exe(request, tmp_path_factory):
    out = str(tmp_path_factory.mktemp("pool") / "pool_fake")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-I", CSRC] +
                   FLAVOURS[request.param] +
                   [os.path.join(ROOT, "tests", "pool_fake.cpp"), "-o", out, "-lpthread"],
                   check=True)
    return out


@pytest.mark.parametrize("scenario", SCENARIOS)
def test_pool(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and scenario + " ok" in r.stdout, r.stdout + r.stderr

"""The integration loop of the table columns (bh_column.h) on the CPU, plain and under
AddressSanitizer + UndefinedBehaviorSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2010_08735_amd", "csrc")
FLAVOURS = {"plain": ["-O2"],
            "asan_ubsan": ["-O2", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=undefined"]}


@pytest.fixture(scope="module", params=list(FLAVOURS))
def exe(request, tmp_path_factory):
    out = str(tmp_path_factory.mktemp("column") / "column_host")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-I", CSRC] +
                   FLAVOURS[request.param] +
                   [os.path.join(ROOT, "tests", "column_host.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("scenario", ["step_limit", "band_rule"])
def test_column(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and scenario + " ok" in r.stdout, r.stdout + r.stderr

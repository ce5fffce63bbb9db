"""Cube faces of area-source probes (bh_probes.h) on the CPU: a tie goes to the lowest axis, also
where the probe's footprint is centred on another face."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_ties_go_to_the_lowest_axis(tmp_path):
    exe = str(tmp_path / "probes_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined", "-I",
                    os.path.join(ROOT, "paper_2010_08735_amd", "csrc"),
                    os.path.join(ROOT, "tests", "probes_host.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr

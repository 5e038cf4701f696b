"""Host check of the plan for the narrow top of circuits with long rows: tests/host_top_check.cpp layerizes random circuits, walks
the streams of every level, and compares a reverse sweep over the levels and the launches' plans below them with one over the
launches' plans alone.  Compiled with the address and undefined-behaviour sanitizers.  No GPU needed."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_levels_and_launches_together_give_the_launches_sweep(tmp_path):
    exe = str(tmp_path / "host_top_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-static-libasan", "-static-libubsan", "-o", exe, os.path.join(ROOT, "tests", "host_top_check.cpp"),
                    os.path.join(ROOT, "paper_2410_11415_amd", "csrc", "layerize.cpp")], check=True, cwd=ROOT)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("ok:"), r.stdout[-2000:] + r.stderr[-2000:]

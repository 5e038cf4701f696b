"""Host check of the units of narrow layers: tests/host_unit_check.cpp cuts random index vectors around the edges of lanes, units and
the limits of rows and layers, and executes the units against sums over the plain index vectors.  Compiled with the address and
undefined-behaviour sanitizers.  No GPU needed."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LAYERIZER = os.path.join(ROOT, "paper_2410_11415_amd", "csrc", "layerize.cpp")


def test_units_hold_every_row_once(tmp_path):
    exe = str(tmp_path / "host_unit_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-static-libasan", "-static-libubsan", "-o", exe, os.path.join(ROOT, "tests", "host_unit_check.cpp"), LAYERIZER],
                   check=True, cwd=ROOT)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("ok:"), r.stdout[-2000:] + r.stderr[-2000:]

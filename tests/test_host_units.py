"""Host checks of the units of narrow layers and of plans without their left-out rows.  tests/host_unit_check.cpp cuts random index
vectors around the edges of lanes, units and
the limits of rows and layers, and executes the units against sums over the plain index vectors; tests/host_compact_check.cpp compares a plan
and the same one with the entries of left-out and split rows taken out.  Compiled with the address and
undefined-behaviour sanitizers.  No GPU needed."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LAYERIZER = os.path.join(ROOT, "paper_2410_11415_amd", "csrc", "layerize.cpp")


@pytest.mark.parametrize("name", ["host_unit_check", "host_compact_check"])
def test_plans_hold_every_row_once(tmp_path, name):
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-static-libasan", "-static-libubsan", "-o", exe, os.path.join(ROOT, "tests", name + ".cpp"), LAYERIZER],
                   check=True, cwd=ROOT)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("ok:"), r.stdout[-2000:] + r.stderr[-2000:]

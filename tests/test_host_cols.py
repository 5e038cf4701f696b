"""Host check of the persistent kernels' streams: tests/host_col_check.cpp cuts random index vectors (rows of 1 to 300000
entries, 1 to 20000 rows) into units and executes the walk of the kernels over them, against sums over the plain index
vectors.  Compiled with the address and undefined-behaviour sanitizers.  No GPU needed."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_units_execute_to_the_plain_sums(tmp_path):
    exe = str(tmp_path / "host_col_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-static-libasan", "-static-libubsan", "-o", exe, os.path.join(ROOT, "tests", "host_col_check.cpp"),
                    os.path.join(ROOT, "paper_2410_11415_amd", "csrc", "layerize.cpp")], check=True, cwd=ROOT)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("ok:"), r.stdout[-2000:] + r.stderr[-2000:]

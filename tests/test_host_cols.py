"""Host check of the persistent kernels' streams: tests/host_col_check.cpp cuts random index vectors (rows of 1 to 300000
entries, 1 to 20000 rows) into units and executes the walk of the kernels over them, against sums over the plain index
vectors.  Compiled with the address and undefined-behaviour sanitizers.  No GPU needed."""
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LAYERIZER = os.path.join(ROOT, "paper_2410_11415_amd", "csrc", "layerize.cpp")


def test_units_execute_to_the_plain_sums(tmp_path):
    exe = str(tmp_path / "host_col_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-static-libasan", "-static-libubsan", "-o", exe, os.path.join(ROOT, "tests", "host_col_check.cpp"), LAYERIZER],
                   check=True, cwd=ROOT)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("ok:"), r.stdout[-2000:] + r.stderr[-2000:]


def test_the_edge_circuits_have_the_runs_they_are_for(tmp_path):
    """what tests/test_gpu_cols.py evaluates with EDGES: layers of the stated sizes whose streams hold, in both directions and for AND
    and OR layers, runs of every kind, of the short kinds with whole blocks and with 0, 1 and 63 rows over a chunk, of the
    long one with units of several blocks"""
    from tests.test_gpu_cols import EDGES, edge_circuit
    exe = str(tmp_path / "host_col_shapes")
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", exe, os.path.join(ROOT, "tests", "host_col_shapes.cpp"), LAYERIZER], check=True, cwd=ROOT)
    seen = {}
    for name, (num_vars, layers) in EDGES.items():
        c = edge_circuit(name)
        path = str(tmp_path / name)
        with open(path, "wb") as f:
            np.array([c.num_vars, c.num_nodes, c.roots.shape[0], c.child_idx.shape[0]], np.int32).tofile(f)
            for a, kind in ((c.node_type, np.uint8), (c.node_lit, np.int32), (c.child_ptr, np.int64), (c.child_idx, np.int32), (c.roots, np.int32)):
                np.ascontiguousarray(a, kind).tofile(f)
        out = subprocess.run([exe, path], capture_output=True, text=True, check=True).stdout.splitlines()
        assert [int(x) for x in out[0].split()] == [2 * num_vars] + [layer[0] for layer in layers]
        for line in out[1:]:
            direction, is_and, kind, k, rows, blocks = map(int, line.split())
            s = seen.setdefault((direction, is_and, kind), dict(full=0, over=set(), quarters=set(), blocks=0))
            per = 1024 >> kind if kind < 3 else 64 >> k
            s["full"] += rows // per
            s["over"].add(rows % 64)
            s["quarters"].add(rows % per * 4 // per)
            s["blocks"] = max(s["blocks"], blocks)
    for direction in (0, 1):
        for is_and in (0, 1):
            for kind in range(5):
                s = seen[direction, is_and, kind]
                if kind < 3:
                    assert s["full"] > 0 and {0, 1, 63} & s["over"] and len(s["quarters"]) > 1, (direction, is_and, kind, s)
            for over in (0, 1, 63):
                assert any(over in seen[direction, is_and, kind]["over"] for kind in range(3)), (direction, is_and, over)
            assert seen[direction, is_and, 3]["blocks"] > 1

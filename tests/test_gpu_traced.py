"""A context that is set up with a profiler attached is the one that is set up
without: the same interior nodes, and so the same bytes a product."""
import os
import shutil
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = """
import sys; sys.path.insert(0, %r)
import torch
from paper_2403_19854_amd import fcrkpm as f, workloads as W
for p in (W.cube(3, 48, 2.5, 1), W.sphere(48, 0.4, 3.0, 2, seed=3)):
    g = f.Problem.from_workload(p, device="cuda:0")
    x = torch.ones(p.shape, device="cuda:0")
    for op in ("K", "M"):
        g.apply(op, x)
        g.profile(True)
        g.apply(op, x)
        g.profile(False)
        print("BYTES", p.name, op, g.profile_read()["tap_k_f32"][2], flush=True)
    g.close()
""" % ROOT


def run(cmd, cwd):
    env = dict(os.environ, TMPDIR=str(cwd))
    r = subprocess.run(cmd, cwd=cwd, env=env, capture_output=True, text=True, timeout=100)
    return [line for line in r.stdout.splitlines() if line.startswith("BYTES")], r


def test_interior_nodes_are_found_under_a_tracer(tmp_path):
    tracer = shutil.which("rocprofv3") or "/opt/rocm/bin/rocprofv3"
    if not os.path.exists(tracer):
        pytest.skip("rocprofv3 is not installed")
    script = tmp_path / "products.py"
    script.write_text(PROGRAM)
    plain, r = run([sys.executable, str(script)], tmp_path)
    assert len(plain) == 4, r.stderr[-2000:]
    traced, r = run([tracer, "--kernel-trace", "-d", str(tmp_path / "out"), "-o", "run", "--output-format", "csv", "--",
                     sys.executable, str(script)], tmp_path)
    if len(traced) < 4:
        pytest.skip("the tracer did not run the program to its end")
    print("\n".join([""] + plain + traced), flush=True)
    assert traced == plain

"""Facts of the planner's results that end results alone would not show (no GPU): memory of a
plan being made."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_python(code):
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout.split()


@pytest.mark.parametrize("n,kmax,gates", [(3, 3, 20000), (2, 2, 20000), (5, 5, 12000)])
def test_planning_a_long_circuit_on_few_qubits_takes_linear_memory(n, kmax, gates):
    """A circuit that fuses into one op is a chain of as many products as gates, each with one
    member more: 128 MiB hold the 64 MiB of products a plan may keep and lists that grow with
    the circuit (tens of MiB), not ones that grow with its square (half a GiB)."""
    out = run_python(f"""
import resource
import numpy as np
from paper_2604_03816_amd import circuits as C, qsv
rng = np.random.default_rng(1)
ops = []
for i in range({gates}):
    q = [int(x) for x in rng.permutation({n})[:2]]
    ops.append(C.Op("CNOT", tuple(q)) if i % 2 else C.Op("RY", (q[0],), (float(rng.uniform(0, 6)),)))
g = qsv.GateList(ops)
before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
p = qsv.Plan({n}, "c128", g, kmax={kmax}, cost_aware=-1)
print(p.stats()["fused_out"], resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before)
""")
    assert int(out[0]) == 1
    assert int(out[1]) <= 128 << 10, out

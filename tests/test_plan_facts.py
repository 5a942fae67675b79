"""Facts of the planner's results that end results alone would not show (no GPU): memory of a
plan being made, what its passes stage, the tables of matrix-core steps, launch limits per device."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2604_03816_amd import build as qsv_build
from paper_2604_03816_amd import circuits as C
from paper_2604_03816_amd import qsv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class PassFacts(ctypes.Structure):   # plan_facts.cpp
    _fields_ = [(f, ctypes.c_int) for f in ("tile_qubits", "low_qubits", "ops", "matrix_ops", "staged", "diag_ops",
                                            "diag_unstaged", "a_len", "d_len", "pool")] + [("tiles", ctypes.c_longlong),
                                                                                           ("pool_total", ctypes.c_longlong)]


@pytest.fixture(scope="module")
def facts(tmp_path_factory):
    qsv.lib()
    so = str(tmp_path_factory.mktemp("plan_facts") / "libplan_facts.so")
    src = os.path.join(ROOT, "tests", "plan_facts.cpp")
    cmd = [qsv_build.HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-fPIC", "-shared",
           "-I" + os.path.join(ROOT, "include"), "-I" + qsv_build.CSRC, "-x", "hip", src, "-o", so,
           "-L" + qsv_build.OUT_DIR, "-lqsv", "-Wl,-rpath," + qsv_build.OUT_DIR]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return ctypes.CDLL(so)


def pass_facts(lib, n, dtype, ops, tile=12):
    g = qsv.GateList(ops)
    out = (PassFacts * 4096)()
    count = lib.plan_facts(n, 0 if dtype == "c64" else 1, tile, g.arr, ctypes.c_size_t(g.n), out, 4096)
    assert 0 <= count <= 4096
    return list(out[:count])


def circuit(name, n, depth, seed):
    if name == "hea":
        return C.bind(C.hea(n, depth), C.hea_params(n, depth, seed))
    return {"brickwork": lambda: C.brickwork(n, depth, seed), "qft": lambda: C.qft(n),
            "bricks": lambda: C.h_t_cz_bricks(n, depth, seed), "mix": lambda: C.commuting_mix(n, 25 * depth, seed)}[name]()


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


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("tile,n,capped", [(12, 15, False), (12, 19, False), (12, 21, False), (12, 23, False), (12, 24, True), (12, 25, True),
                                           (11, 25, False), (10, 22, False)])
def test_operands_end_a_pass_only_where_it_may_load_ahead(facts, dtype, tile, n, capped):
    """A pass on tiles of 2^12 amplitudes whose launch covers 2^13 of them (two states count
    twice) loads its next tile during the ops if all matrix operands are in LDS, so the planner
    ends it where they are full; on other tiles and below, one with more operands is as good."""
    fs = pass_facts(facts, n, dtype, C.brickwork(n, 8, 3), tile)
    assert all(f.tile_qubits == tile and f.tiles == 1 << (n - tile) for f in fs)
    assert all(f.staged for f in fs) == capped


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("name,depth", [("hea", 6), ("hea", 12), ("qft", 1), ("bricks", 12), ("mix", 12), ("brickwork", 8)])
def test_passes_that_load_ahead_have_their_matrix_operands_staged(facts, name, depth, dtype):
    """Whatever diagonal tables share the pass's block in LDS."""
    for n in range(25, 31):
        for p, f in enumerate(pass_facts(facts, n, dtype, circuit(name, n, depth, 1))):
            assert f.staged, (n, p, f.matrix_ops, f.diag_ops, f.a_len)
            assert f.d_len <= f.a_len <= (2048 if dtype == "c64" else 4096)


@pytest.mark.parametrize("n,steps", [(14, 28), (15, 28), (16, 30), (17, 34), (18, 36), (19, 38)])
def test_few_tiles_save_passes_and_steps(facts, n, steps):
    """complex64 states with fewer tiles than CUs: the 8-layer ansatz needs no more passes than
    with its operands capped (6 to 9), and no diagonal steps bought with them."""
    fs = pass_facts(facts, n, "c64", circuit("hea", n, 8, 1))
    assert len(fs) <= n // 2 - 1 and sum(f.ops for f in fs) <= steps


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("name,n,depth", [("brickwork", 20, 8), ("hea", 18, 6), ("mix", 16, 12), ("brickwork", 6, 4)])
def test_the_pool_holds_what_ops_read_and_no_more(facts, name, n, depth, dtype):
    """Matrix-core ops read their operands; their matrices are not carried a second time."""
    fs = pass_facts(facts, n, dtype, circuit(name, n, depth, 2))
    assert sum(f.pool for f in fs) == fs[0].pool_total


def test_launch_limits_are_raised_once_on_each_device(facts):
    """A kernel's dynamic LDS limit belongs to a device: the step runs once on each, again where
    it failed, and always beyond the 64 devices that are kept apart."""
    devices = [0, 0, 1, 1, 0, 2, 1, 63, 63, 64, 64]
    ran = (ctypes.c_int * len(devices))()
    assert facts.runs_per_device((ctypes.c_int * len(devices))(*devices), len(devices), 2, ran) == 1
    assert list(ran) == [1, 0, 1, 1, 0, 1, 0, 1, 0, 1, 1]


@pytest.mark.parametrize("forward,undo,plans,want", [
    (100 << 10, 30 << 10, 72, (8, 100 << 10)),      # many plans: every slot
    (100 << 10, 30 << 10, 3, (3, 100 << 10)),       # a short circuit, one vector
    (100 << 10, 0, 1, (0, 0)),                      # one plan: its slot grows when it comes
    (2 << 20, 1 << 10, 80, (8, 2 << 20)), ((2 << 20) + 1, 1 << 10, 80, (8, 1 << 10)),   # a deep circuit
    (40 << 20, 3 << 20, 80, (0, 0)), (40 << 20, 3 << 20, 5, (5, 3 << 20)), (1000, 999, 2, (2, 1024))])
def test_a_gradient_call_reserves_what_its_plans_take(facts, forward, undo, plans, want):
    b = ctypes.c_size_t()
    facts.reserved_slots.argtypes = [ctypes.c_size_t] * 3 + [ctypes.c_int, ctypes.POINTER(ctypes.c_size_t)]
    got = facts.reserved_slots(forward, undo, plans, 8, ctypes.byref(b))
    assert (got, b.value) == want


def random_dense(n, count, seed):
    rng = np.random.default_rng(seed)
    ops = []
    for _ in range(count):
        k = int(rng.choice([2, 3, 3, 4, 4, 4]))
        ops.append(C.Op("U", tuple(int(q) for q in rng.permutation(n)[:k]), matrix=C.haar_unitary(rng, 1 << k)))
    return ops


@pytest.mark.parametrize("dtype,tol", [("c64", 1e-5), ("c128", 1e-13)])
@pytest.mark.parametrize("tile,n", [(8, 8), (8, 14), (9, 9), (10, 10), (10, 16), (11, 16), (12, 12), (12, 20), (13, 15)])
def test_matrix_core_steps_from_their_tables(facts, tile, n, dtype, tol):
    """Operand and offset tables walked lane by lane: every tile slot read and written once by
    one wave, no barrier left out where a wave would read another's slots, and the product the
    gates' own (entries rounded to the state's precision: 2^-24 of sums of 16 terms of size 1.4,
    twice in a pair, stays under 1e-5; FP64 under 1e-13)."""
    if dtype == "c128" and tile > 12:
        pytest.skip("13-qubit tiles fit LDS only in complex64")
    facts.check_steps.argtypes = [ctypes.c_int] * 3 + [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int,
                                                       ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_int)]
    free = 0
    for seed in range(4):
        for ops in (random_dense(n, 40, seed), circuit("hea", n, 4, seed), circuit("brickwork", n, 6, seed)):
            g, worst, nosync = qsv.GateList(ops), ctypes.c_double(), ctypes.c_int()
            steps = facts.check_steps(n, 0 if dtype == "c64" else 1, tile, g.arr, g.n, seed < 2, ctypes.byref(worst),
                                      ctypes.byref(nosync))
            assert steps > 0 and worst.value <= tol, (seed, steps, worst.value)
            free += nosync.value
    assert (free > 0) == (tile >= 10)

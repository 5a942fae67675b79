"""Matrix-core ops (libqsv, through the C ABI) against the FP64 oracle where their tables and
launches change shape: one tile and many, tiles taken one or several per workgroup (the
next one loaded ahead), ops run alone, as pairs on disjoint targets, behind diagonal ops and
permutations, and with and without a barrier between neighbours.  Tolerances are the parity
bars: max|d alpha| <= 1e-12 (complex128), <= 5e-6 (complex64)."""
import numpy as np
import pytest

import oracle
from paper_2604_03816_amd import circuits as C

pytestmark = pytest.mark.gpu
TOL = {"c128": 1e-12, "c64": 5e-6}


def dense(rng, qubits):
    return C.Op("U", tuple(int(q) for q in qubits), matrix=C.haar_unitary(rng, 1 << len(qubits)))


def matrix_circuit(n, rng):
    """4- and 3-qubit dense ops on neighbouring, disjoint, overlapping and scattered targets."""
    hi = n - 1
    ops = [dense(rng, (0, 1, 2, 3)), dense(rng, (4, 5, 6, 7)),       # a pair
           dense(rng, (2, 3, 4, 5)),                                 # overlaps both
           dense(rng, (hi, hi - 1, hi - 2)), dense(rng, (0, 3, 5)),  # 3-qubit, disjoint when n > 8
           dense(rng, (1, 6, hi, 4))]
    ops.append(C.Op("U", (0, hi), matrix=np.diag(np.exp(1j * rng.uniform(0, 6, 4)))))
    ops.append(C.Op("CNOT", (hi, 1)))
    for _ in range(4):
        qs = rng.permutation(n)
        ops += [dense(rng, qs[:4]), dense(rng, qs[4:8])]             # a pair on any qubits
        ops.append(dense(rng, rng.permutation(n)[:3]))
    return ops


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [8, 9, 12, 13, 14, 19, 25])
def test_matrix_core_ops(dtype, n):
    from paper_2604_03816_amd import qsv
    ops = matrix_circuit(n, np.random.default_rng(100 + n))
    s = qsv.State(n, dtype)
    plan = qsv.Plan(n, dtype, ops, kmax=4)
    assert plan.stats()["mfma_ops"] > 0
    ref = oracle.simulate(n, ops)
    s.apply_plan(plan)
    assert oracle.max_abs_diff(ref, s.get()) <= TOL[dtype]
    s.apply_plan_zero(plan)
    assert oracle.max_abs_diff(ref, s.get()) <= TOL[dtype]
    s.free()


@pytest.mark.parametrize("tile", [8, 10, 13])
def test_matrix_core_ops_on_other_tiles(tile):
    from paper_2604_03816_amd import qsv
    n = 16
    ops = matrix_circuit(n, np.random.default_rng(7))
    ref = oracle.simulate(n, ops)
    for dtype in ("c64", "c128"):
        if dtype == "c128" and tile > 12:
            continue
        s = qsv.State(n, dtype)
        s.apply(ops, kmax=4, tile_qubits=tile, low_qubits=2)
        assert oracle.max_abs_diff(ref, s.get()) <= TOL[dtype]
        s.free()


def test_split_products_keep_small_and_large_amplitudes():
    """complex64 products through exact splits hold small amplitudes beside large ones: a
    block-diagonal op keeps a column scaled by 2^-40 at the accuracy of its own size."""
    from paper_2604_03816_amd import qsv
    n = 12
    rng = np.random.default_rng(3)
    u = np.zeros((16, 16), complex)
    u[:8, :8], u[8:, 8:] = C.haar_unitary(rng, 8), C.haar_unitary(rng, 8)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi = (psi / np.linalg.norm(psi)).astype(np.complex64)
    small = (np.arange(1 << n) >> 5 & 1) == 1      # the op's local bit 3 is qubit 5
    psi[small] *= np.float32(2.0 ** -40)
    s = qsv.State(n, "c64")
    s.set(psi)
    ops = [C.Op("U", (2, 3, 4, 5), matrix=u)]
    s.apply(ops, kmax=4)
    ref = psi.astype(np.complex128)
    oracle.apply(ref, u, (2, 3, 4, 5))
    got = s.get()
    scale = np.abs(ref[small]).max()
    # eight products of rounded entries (2^-24) summed in FP32: well below 2^-19 of the largest
    assert np.max(np.abs(got[small] - ref[small])) <= 2.0 ** -19 * scale
    s.free()


@pytest.mark.parametrize("k,targets", [(4, (2, 3, 4, 5)), (3, (1, 5, 9))])
def test_the_range_of_split_products(k, targets):
    """complex64 states of sizes over the range in which splits are exact, and beyond it (and
    with an infinity) with matrix_cores = -1.  The bound is the one above: 2^-19 of the largest."""
    from paper_2604_03816_amd import qsv
    n = 12
    rng = np.random.default_rng(5)
    u = C.haar_unitary(rng, 1 << k)
    psi0 = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi0 /= 2 * np.abs(psi0).max()
    s = qsv.State(n, "c64")
    for e, opts in ((0, {}), (-60, {}), (-100, {}), (100, {}), (125, {}), (-118, {"matrix_cores": -1}),
                    (125, {"matrix_cores": -1})):
        psi = (psi0 * 2.0 ** e).astype(np.complex64)
        s.set(psi)
        s.apply([C.Op("U", targets, matrix=u)], kmax=4, **opts)
        ref = psi.astype(np.complex128)
        oracle.apply(ref, u, targets)
        assert np.max(np.abs(s.get() - ref)) <= 2.0 ** -19 * np.abs(ref).max(), (e, opts)
    psi = psi0.astype(np.complex64)
    psi[77] = np.inf
    bits = sum(1 << t for t in targets)
    group = (np.arange(1 << n) & ~bits) == 77 & ~bits
    for opts, most in (({}, 16), ({"matrix_cores": -1}, 1 << k)):
        s.set(psi)
        s.apply([C.Op("U", targets, matrix=u)], kmax=4, **opts)
        got = s.get()
        bad = ~np.isfinite(got)
        assert np.all(bad[group]) and bad.sum() <= most
        ref = np.where(group, 0, psi).astype(np.complex128)
        oracle.apply(ref, u, targets)
        assert np.max(np.abs(got[~bad] - ref[~bad])) <= 2.0 ** -19
    s.free()

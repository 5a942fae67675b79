"""Marginal distributions against the FP64 oracle around the block kernel's edges: states of one
small block, one full block and many; measured qubits inside, above and across the block's
bits, one to all but one of them, in any order; one and several workgroups per value of the
measured qubits above.  Every entry is a compensated FP64 sum: 1e-14."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 5, 11, 12, 13, 16, 20])
def test_marginals(dtype, n):
    import torch
    from paper_2604_03816_amd import qsv
    rng = np.random.default_rng(n)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi /= np.linalg.norm(psi)
    s = qsv.State(n, dtype)
    s.set(psi)
    ref = s.get().astype(np.complex128)
    sets = [(0,), (n - 1,), tuple(range(n))[::-1], tuple(range(0, n, 2)), tuple(range(min(n, 12)))[::-1]]
    sets += [tuple(range(12, n))] if n > 12 else []
    for m in sorted({1, 2, n // 3, n // 2, n - 2, n - 1}):
        if m >= 1:
            sets.append(tuple(int(q) for q in rng.permutation(n)[:m]))
    for qubits in sets:
        if list(qubits) == list(range(n)):
            continue   # the full distribution
        want = oracle.probs(ref, list(qubits))
        got = s.probs(qubits)
        assert got.dtype == np.float64 and np.max(np.abs(got - want)) <= 1e-14, qubits
        out = torch.empty(1 << len(qubits), dtype=torch.float64, device="cuda:0")
        assert np.array_equal(s.probs(qubits, out=out).cpu().numpy(), got), qubits
    s.free()

"""Timed workloads of the framework: what a program that uses it has it do.

Each case is a dict of plain values.  `kind` names the entry points a case goes through:

  step     a kept plan applied to |0...0>, then the norm and a Pauli sum (the simulation
           step of `bench.py`, and one energy of a variational program)
  apply    a circuit given as gates: planned, fused and applied in one call, then a Pauli sum
  observe  Pauli sums with X, Y and Z factors, the norm and marginal distributions of a state
  sample   measurement outcomes of a state
  grad     energies and gradients of a parameterised circuit (autograd, forward + backward)
  noise    a circuit with noise channels on a density matrix, its distribution and a Pauli sum
  serve    a batch of requests through the continuous-batching server

`dtype` is the state's: "c64" or "c128".  Values derived from a complex64 state are returned
in float32, the precision they have.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2604_03816_amd import autograd, circuits, qsv, serve

DEVICE = "cuda:0"


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the smallest circuits (the smoke test's size): a call's latency
        {"name": "step brickwork 10 c64", "kind": "step", "circuit": "brickwork", "n": 10, "depth": 20, "dtype": "c64"},
        # an energy of a variational program at an ordinary size
        {"name": "step hea 18 c128", "kind": "step", "circuit": "hea", "n": 18, "depth": 6, "dtype": "c128"},
        # gates on arbitrary qubits, many of them diagonal or controlled, at an odd size
        {"name": "step mix 25 c64", "kind": "step", "circuit": "mix", "n": 25, "depth": 12, "dtype": "c64"},
        # the benchmark's circuit at its size, and the fusion study's in double precision
        {"name": "step brickwork 30 c64", "kind": "step", "circuit": "brickwork", "n": 30, "depth": 20, "dtype": "c64"},
        {"name": "step brickwork 28 c128", "kind": "step", "circuit": "brickwork", "n": 28, "depth": 20,
         "dtype": "c128"},
        # a circuit given once (QFT-20), planned and applied in one call
        {"name": "apply qft 20 c128", "kind": "apply", "circuit": "qft", "n": 20, "depth": 1, "dtype": "c128"},
        # the observables of a state that a program holds
        {"name": "observe 27 c64", "kind": "observe", "n": 27, "dtype": "c64", "terms": 80, "marginal": 5},
        # 2^20 shots of a state
        {"name": "sample 28 c64", "kind": "sample", "n": 28, "dtype": "c64", "shots": 1 << 20, "marginal": 0},
        # gradients: a batch of small circuits, and a large circuit (the gradient workload's ansatz)
        {"name": "grad 12 c128", "kind": "grad", "n": 12, "depth": 4, "batch": 8, "dtype": "c128"},
        {"name": "grad 22 c64", "kind": "grad", "n": 22, "depth": 8, "batch": 2, "dtype": "c64"},
        # the noise study's model on a layered circuit
        {"name": "noise 11 c128", "kind": "noise", "n": 11, "depth": 6, "dtype": "c128"},
        # requests of the serving stream's shape, all waiting
        {"name": "serve 96", "kind": "serve", "requests": 96, "n_hi": 23, "d_hi": 60, "dtype": "mixed"},
    ]


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["apply", "observe", "sample", "grad", "grad", "noise", "serve"])
    dtype = rng.choice(["c64", "c128"])
    wide = dtype == "c128"
    if kind == "step":
        return {"kind": kind, "circuit": rng.choice(["brickwork", "hea", "mix", "qft", "bricks", "random1q"]),
                "n": rng.randint(8, 28 if wide else 29), "depth": rng.randint(4, 20), "dtype": dtype}
    if kind == "apply":
        return {"kind": kind, "circuit": rng.choice(["brickwork", "hea", "mix", "qft", "bricks", "random1q"]),
                "n": rng.randint(6, 25), "depth": rng.randint(2, 12), "dtype": dtype}
    if kind == "observe":
        return {"kind": kind, "n": rng.randint(8, 27 if wide else 28), "dtype": dtype, "terms": rng.randint(5, 120),
                "marginal": rng.randint(1, 8)}
    if kind == "sample":
        return {"kind": kind, "n": rng.randint(10, 27 if wide else 28), "dtype": dtype,
                "shots": int(2 ** rng.uniform(10, 20)), "marginal": rng.choice([0, 0, rng.randint(1, 9)])}
    if kind == "grad":
        return {"kind": kind, "n": rng.randint(6, 22), "depth": rng.randint(2, 8), "batch": rng.randint(1, 4),
                "dtype": dtype}
    if kind == "noise":
        return {"kind": kind, "n": rng.randint(3, 12), "depth": rng.randint(2, 8), "dtype": dtype}
    return {"kind": kind, "requests": rng.randint(16, 96), "n_hi": rng.randint(16, 23), "d_hi": rng.randint(20, 60),
            "dtype": "mixed"}


# ------------------------------------------------------------------ inputs

def _ops(case, seed):
    """The case's circuit; `depth` counts layers (mix: 25 gates a layer)."""
    n, d, c = case["n"], case["depth"], case["circuit"]
    if c == "brickwork":
        return circuits.brickwork(n, d, seed)
    if c == "hea":
        return circuits.bind(circuits.hea(n, d), circuits.hea_params(n, d, seed))
    if c == "mix":
        return circuits.commuting_mix(n, 25 * d, seed)
    if c == "bricks":
        return circuits.h_t_cz_bricks(n, d, seed)
    if c == "random1q":
        return circuits.random_1q(n, seed, gates_per_qubit=d)
    # the QFT of a product state with an angle per qubit from the seed
    th = np.random.default_rng(seed).uniform(0.0, 2.0 * math.pi, n)
    return [circuits.Op("RY", (q,), (float(th[q]),)) for q in range(n)] + circuits.qft(n)


def _noisy(case, seed):
    """Layers of rotations and CNOT bricks, each gate followed by depolarizing noise, with
    amplitude damping at the end."""
    n = case["n"]
    rng = np.random.default_rng(seed)
    ops = [circuits.Op("H", (0,))]
    for layer in range(case["depth"]):
        for q in range(n):
            ops.append(circuits.Op("RY", (q,), (float(rng.uniform(0.0, 2.0 * math.pi)),)))
        for q in range(layer % 2, n - 1, 2):
            ops.append(circuits.Op("CNOT", (q, q + 1)))
    ops = circuits.with_depolarizing(ops, 0.002, 0.01)
    return ops + [circuits.Op("AMPDAMP", (q,), (0.02,)) for q in range(n)]


def _terms(case, seed):
    """Z chains, single X, XX and YY pairs and a few longer strings."""
    n = case["n"]
    rng = np.random.default_rng(seed)
    terms = []
    for t in range(case["terms"]):
        r, c, q = t % 4, float(rng.normal()), int(rng.integers(0, n - 1))
        if r == 0:
            terms.append((c, ((q, "Z"), (q + 1, "Z"))))
        elif r == 1:
            terms.append((c, ((q, "X"),)))
        elif r == 2:
            p = "XY"[t // 4 % 2]
            terms.append((c, ((q, p), (q + 1, p))))
        else:
            qs = rng.permutation(n)[: min(n, 4)]
            terms.append((c, tuple((int(x), "XYZZ"[i]) for i, x in enumerate(qs))))
    return terms


def _random_state(n, dtype, seed):
    """A random state's amplitudes (what a deep circuit leaves), normalised."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    tdt = torch.complex64 if dtype == "c64" else torch.complex128
    t = torch.randn(1 << n, dtype=tdt, device=DEVICE, generator=g)
    return t.mul_(1.0 / math.sqrt(2.0 ** n))


def _requests(case, seed):
    """The serving stream's sizes and precisions; the seed draws the circuits' gates."""
    reqs = circuits.serving_stream(case["requests"], n_hi=case["n_hi"], d_hi=case["d_hi"])
    return [dataclasses.replace(r, seed=r.seed + seed) for r in reqs]


def _qubits(case, seed):
    m = min(case["marginal"], case["n"])
    return [int(q) for q in np.random.default_rng(seed + 1).permutation(case["n"])[:m]] if m else None


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "kind": kind, "f32": case["dtype"] == "c64"}
    if kind == "step":
        st["plan"] = qsv.Plan(case["n"], case["dtype"], _ops(case, seed))
        st["state"] = qsv.State(case["n"], case["dtype"])
        st["terms"] = qsv.TermList(circuits.tfim_terms(case["n"]))
    elif kind == "apply":
        st["gates"] = qsv.GateList(_ops(case, seed))
        st["state"] = qsv.State(case["n"], case["dtype"])
        st["terms"] = qsv.TermList(circuits.tfim_terms(case["n"]))
    elif kind in ("observe", "sample"):
        st["state"] = qsv.State(case["n"], case["dtype"])
        st["state"].tensor.copy_(_random_state(case["n"], case["dtype"], seed))
        if kind == "observe":
            st["terms"] = qsv.TermList(_terms(case, seed))
        else:
            st["uniforms"] = np.random.default_rng(seed).random(case["shots"])
        st["qubits"] = _qubits(case, seed)
    elif kind == "grad":
        st["template"] = qsv.OpList(circuits.hea(case["n"], case["depth"], ring=True))
        st["terms"] = qsv.TermList(circuits.tfim_terms(case["n"]))
        p = circuits.hea_params(case["n"], case["depth"], seed, batch=case["batch"])
        st["params"] = torch.tensor(p, dtype=torch.float32 if st["f32"] else torch.float64, requires_grad=True)
    elif kind == "noise":
        st["ops"] = qsv.DMOpList(_noisy(case, seed))
        st["rho"] = qsv.DensityMatrix(case["n"], case["dtype"])
        st["terms"] = qsv.TermList(circuits.tfim_terms(case["n"]))
    else:
        reqs = _requests(case, seed)
        st["requests"] = reqs
        st["gates"] = [qsv.ArrayGateList(circuits.brickwork_arrays(r.n, r.depth, r.seed)) for r in reqs]
        st["server"] = serve.Server(max_slots=64, use_graph=True)
    return st


# ------------------------------------------------------------------ one pass

def run(st):
    kind = st["kind"]
    real = (lambda v: np.asarray(v, dtype=np.float32)) if st["f32"] else np.asarray
    if kind == "step":
        s = st["state"]
        s.apply_plan_zero(st["plan"])
        norm = s.norm()
        _, per = s.expval(st["terms"], per_term=True)
        return {"state": s.tensor, "norm": real(norm), "terms": real(per)}
    if kind == "apply":
        s = st["state"]
        s.reset()
        s.apply(st["gates"])
        _, per = s.expval(st["terms"], per_term=True)
        return {"state": s.tensor, "terms": real(per)}
    if kind == "observe":
        s = st["state"]
        e, per = s.expval(st["terms"], per_term=True)
        return {"sum": e, "terms": per, "norm": s.norm(), "marginal": s.probs(st["qubits"])}
    if kind == "sample":
        return st["state"].sample(st["uniforms"], st["qubits"])
    if kind == "grad":
        p = st["params"]
        p.grad = None
        e = autograd.expval(p, st["case"]["n"], st["template"], st["terms"], st["case"]["dtype"])
        e.sum().backward()
        return {"energy": e.detach(), "grad": p.grad}
    if kind == "noise":
        rho = st["rho"]
        rho.reset()
        rho.apply(st["ops"])
        _, per = rho.expval(st["terms"], per_term=True)
        return {"rho": rho.state.tensor, "probs": real(rho.probs()), "terms": real(per)}
    sv, reqs = st["server"], st["requests"]
    at = {sv.submit(r.n, r.dtype, g): i for i, (r, g) in enumerate(zip(reqs, st["gates"]))}
    got = [None] * len(reqs)
    left = len(reqs)
    while left:
        sv.step()
        for res in sv.results():
            got[at[res["id"]]] = res
            left -= 1
    single = [np.append(r["zexp"], r["norm"]) for r in got if r["dtype"] == "c64"]
    double = [np.append(r["zexp"], r["norm"]) for r in got if r["dtype"] == "c128"]
    return {"single": np.concatenate(single).astype(np.float32), "double": np.concatenate(double)}


# ------------------------------------------------------------------ what a pass cannot do without

def _gate_flops(k, named):
    """Real operations per amplitude of one gate: a dense one takes 2^k complex
    multiply-adds, a permutation none, a phase one complex multiply."""
    if named in ("CNOT", "SWAP", "TOFFOLI", "X"):
        return 0
    if named in ("CZ", "RZ", "T", "S", "Z", "phase"):
        return 6
    return 8 << k


def _circuit_flops(case):
    return sum(_gate_flops(len(op.qubits), op.name if op.matrix is None or np.count_nonzero(op.matrix) > len(op.matrix)
                           else "phase") for op in _ops(case, 1))


def work(case):
    kind, elem = case["kind"], 8 if case["dtype"] == "c64" else 16
    if kind in ("step", "apply"):
        amps = 2.0 ** case["n"]
        return {"bytes": amps * elem, "flops": amps * (_circuit_flops(case) + 4 + 8 * 2 * case["n"])}
    if kind == "observe":
        amps = 2.0 ** case["n"]
        return {"bytes": amps * elem, "flops": amps * (4 + 8 * case["terms"])}
    if kind == "sample":
        return {"bytes": 2.0 ** case["n"] * elem + 16.0 * case["shots"], "flops": 4.0 * 2.0 ** case["n"]}
    if kind == "grad":
        n, layers = case["n"], case["depth"]
        per_layer = n * (_gate_flops(1, "RY") + 6) + n * 6
        # forward once, then both states undone, and one element per parameter
        return {"bytes": case["batch"] * 16.0 * (2 * n * layers + 1),
                "flops": case["batch"] * 2.0 ** n * (3.0 * layers * per_layer + 8 * 2 * n * layers + 8 * 2 * n)}
    if kind == "noise":
        amps = 4.0 ** case["n"]
        flops = 0
        for op in _noisy(case, 1):
            k = len(op.qubits)
            flops += 8 << (2 * k) if op.name in circuits.CHANNELS else 2 * _gate_flops(k, op.name)
        return {"bytes": amps * elem, "flops": amps * flops}
    byts = flops = 0.0
    for r in _requests(case, 1):
        byts += 8.0 * (r.n + 1)
        flops += 2.0 ** r.n * (16.0 * r.n * r.depth + 2 * r.n)
    return {"bytes": byts, "flops": flops}


# ------------------------------------------------------------------ the same in 64 bits

def _op_matrix(op):
    """An op's matrix from its definition (local bit j <-> qubits[j])."""
    if op.matrix is not None:
        return np.asarray(op.matrix, dtype=np.complex128)
    if op.name in ("RX", "RY", "RZ"):
        t = op.params[0]
        p = {"RX": [[0, 1], [1, 0]], "RY": [[0, -1j], [1j, 0]], "RZ": [[1, 0], [0, -1]]}[op.name]
        return math.cos(t / 2) * np.eye(2) - 1j * math.sin(t / 2) * np.array(p, dtype=np.complex128)
    if op.name == "H":
        return np.array([[1, 1], [1, -1]], dtype=np.complex128) / math.sqrt(2.0)
    if op.name == "T":
        return np.diag([1, complex(math.sqrt(0.5), math.sqrt(0.5))])
    d = {"CNOT": 4, "CZ": 4, "TOFFOLI": 8}[op.name]
    m = np.zeros((d, d), dtype=np.complex128)
    for i in range(d):
        j = i ^ 2 if op.name == "CNOT" and i & 1 else i ^ 4 if op.name == "TOFFOLI" and i & 3 == 3 else i
        m[j, i] = -1 if op.name == "CZ" and i == 3 else 1
    return m


def _act(psi, m, qubits):
    """The matrix `m` on `qubits` of the vector psi (any length 2^n), out of place."""
    k = len(qubits)
    order = sorted(range(k), key=lambda j: -qubits[j])   # highest qubit first
    shape, prev = [], psi.numel().bit_length() - 1
    for j in order:
        shape += [1 << (prev - qubits[j] - 1), 2]
        prev = qubits[j]
    v = psi.view(shape + [1 << prev])
    out = torch.empty_like(v)

    def row(t, r):
        for a, j in enumerate(order):
            t = t.select(2 * a + 1 - a, (r >> j) & 1)
        return t

    for r in range(1 << k):
        to = row(out, r)
        cols = [c for c in range(1 << k) if m[r, c] != 0]
        if not cols:
            to.zero_()
        for i, c in enumerate(cols):
            if i == 0:
                torch.mul(row(v, c), complex(m[r, c]), out=to)
            else:
                to.add_(row(v, c), alpha=complex(m[r, c]))
    return out.view(-1)


def _zero(n):
    psi = torch.zeros(1 << n, dtype=torch.complex128, device=DEVICE)
    psi[0] = 1
    return psi


def _simulate(n, ops):
    psi = _zero(n)
    for op in ops:
        psi = _act(psi, _op_matrix(op), op.qubits)
    return psi


_PAULI = {"X": np.array([[0, 1], [1, 0]]), "Y": np.array([[0, -1j], [1j, 0]]), "Z": np.array([[1, 0], [0, -1]])}


def _pauli_act(psi, string):
    for q, p in string:
        psi = _act(psi, _PAULI[p].astype(np.complex128), (q,))
    return psi


def _expvals(psi, terms):
    return np.array([c * torch.vdot(psi, _pauli_act(psi, s)).real.item() for c, s in terms])


def _norm2(psi):
    return torch.view_as_real(psi).square().sum().item()


def _exact_grad(case, seed):
    n = case["n"]
    params = circuits.hea_params(n, case["depth"], seed, batch=case["batch"])
    if case["dtype"] == "c64":
        params = params.astype(np.float32).astype(np.float64)
    terms = circuits.tfim_terms(n)
    axis = {"RX": "X", "RY": "Y", "RZ": "Z"}
    E, G = np.zeros(len(params)), np.zeros_like(params)
    for b, p in enumerate(params):
        ops = circuits.bind(circuits.hea(n, case["depth"], ring=True), p)
        psi = _simulate(n, ops)
        lam = torch.zeros_like(psi)
        for c, s in terms:
            lam += c * _pauli_act(psi, s)
        E[b] = torch.vdot(psi, lam).real.item()
        for op in reversed(ops):
            if op.param is not None:
                G[b, op.param] += torch.vdot(lam, _pauli_act(psi, ((op.qubits[0], axis[op.name]),))).imag.item()
            m = _op_matrix(op).conj().T
            psi, lam = _act(psi, m, op.qubits), _act(lam, m, op.qubits)
    return {"energy": torch.from_numpy(E), "grad": torch.from_numpy(G)}


def _exact_noise(case, seed):
    n = case["n"]
    rho = _zero(2 * n)   # entry [row, col] at row + 2^n col
    for op in _noisy(case, seed):
        q = op.qubits
        if op.name == "AMPDAMP":
            g = op.params[0]
            kraus = [np.diag([1, math.sqrt(1 - g)]).astype(complex), np.array([[0, math.sqrt(g)], [0, 0]], complex)]
        elif op.name == "DEPOLARIZE":
            strings = [np.eye(1, dtype=complex)]
            for _ in q:
                strings = [np.kron(a, b) for a in strings for b in [np.eye(2)] + [_PAULI[x] for x in "XYZ"]]
            p = op.params[0]
            w = [1 - p] + [p / (len(strings) - 1)] * (len(strings) - 1)
            kraus = [math.sqrt(x) * s for x, s in zip(w, strings)]
        else:
            m = _op_matrix(op)
            rho = _act(_act(rho, m, q), m.conj(), tuple(t + n for t in q))
            continue
        rho = _act(rho, sum(np.kron(k.conj(), k) for k in kraus), q + tuple(t + n for t in q))
    v = rho.view(1 << n, 1 << n)   # [col, row]
    per = []
    for c, s in circuits.tfim_terms(n):
        d = rho
        for t, p in s:
            d = _act(d, _PAULI[p].astype(complex), (t,))   # P rho
        per.append(c * d.view(1 << n, 1 << n).diagonal().real.sum().item())
    return {"rho": rho, "probs": v.diagonal().real.contiguous(), "terms": np.array(per)}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "apply"):
        if case["n"] > 26:
            return None   # more than 20 seconds
        psi = _simulate(case["n"], _ops(case, seed))
        got = {"state": psi, "terms": _expvals(psi, circuits.tfim_terms(case["n"]))}
        if kind == "step":
            got["norm"] = np.asarray(_norm2(psi))
        return got
    if kind == "observe":
        psi = _random_state(case["n"], case["dtype"], seed).to(torch.complex128)
        per = _expvals(psi, _terms(case, seed))
        p = torch.view_as_real(psi).square().sum(-1)
        qubits = _qubits(case, seed)
        shape, prev, kept = [], case["n"], []
        for q in sorted(qubits, reverse=True):
            shape += [1 << (prev - q - 1), 2]
            prev = q
            kept.append(q)
        p = p.view(shape + [1 << prev]).sum(dim=tuple(range(0, 2 * len(kept) + 1, 2)))
        # axes now go from the highest measured qubit down; the output's bit j is qubits[j]
        p = p.permute([kept.index(q) for q in reversed(qubits)]).reshape(-1)
        return {"sum": math.fsum(per), "terms": per, "norm": _norm2(psi), "marginal": p.cpu().numpy()}
    if kind == "grad":
        return _exact_grad(case, seed)
    if kind == "noise":
        return _exact_noise(case, seed)
    if kind == "serve":
        single, double = [], []
        for r in _requests(case, seed):
            psi = _simulate(r.n, circuits.brickwork(r.n, r.depth, r.seed))
            p = torch.view_as_real(psi).square().sum(-1)
            norm = p.sum().item()
            z = [norm - 2.0 * p.view(-1, 2, 1 << q)[:, 1].sum().item() for q in range(r.n)]
            (single if r.dtype == "c64" else double).extend(z + [norm])
        return {"single": np.array(single), "double": np.array(double)}
    return None   # outcomes are whole numbers

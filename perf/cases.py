"""Performance cases: circuit batches as a user's program runs them.

Every case is one call (or one training step) of the public binding
``paper_2003_02989_amd.tq`` on a circuit family that the repository's
workloads, tests and benchmark use: hardware-efficient ansatz, QNN classifier,
QAOA MaxCut, random grid circuits, the VQE ansatz with its Pauli Hamiltonian
(exact, from measurement shots, and noisy), and ragged batches of different
circuits.  ``prepare`` holds what such a program keeps (program, observables,
symbol values); ``exact`` computes the same outputs in complex128 with plain
torch, gate by gate.
"""
import math
import random

import numpy as np
import torch

from paper_2003_02989_amd import tq
from paper_2003_02989_amd.circuits import Circuit, const, observable_blob, program_blob, sym


def listed():
    return [
        # policy / PQC training step on a handful of tiny circuits: all latency
        {"name": "hea_n4_b16_adjoint", "family": "hea", "call": "adjoint", "n": 4, "batch": 16, "layers": 2},
        # training step of the QNN classifier on one batch of encoded inputs
        {"name": "qnn_n10_b1024_adjoint", "family": "qnn", "call": "adjoint", "n": 10, "batch": 1024, "layers": 4},
        # the same classifier trained with hardware's gradient rule
        {"name": "qnn_n10_b256_shift", "family": "qnn", "call": "param_shift", "n": 10, "batch": 256, "layers": 4},
        # QAOA MaxCut: cost of a population of angle sets
        {"name": "qaoa_n20_b256_cost", "family": "qaoa", "call": "expectation", "n": 20, "batch": 256, "layers": 4},
        # QAOA gradients by the shift rule on a mid-sized graph
        {"name": "qaoa_n14_b24_shift", "family": "qaoa", "call": "param_shift", "n": 14, "batch": 24, "layers": 3},
        # amplitudes of the 30-qubit random circuit: the largest state
        {"name": "grid_n30_amplitudes", "family": "grid", "call": "samples", "n": 30, "rows": 5, "depth": 20,
         "batch": 1, "shots": 0, "bitstrings": 4096},
        # samples and amplitudes of a smaller random circuit
        {"name": "grid_n24_samples", "family": "grid", "call": "samples", "n": 24, "rows": 4, "depth": 14,
         "batch": 1, "shots": 200000, "bitstrings": 1000},
        # VQE: a full training step over many parameter sets, 200 Pauli strings
        {"name": "vqe_n16_b4096_adjoint", "family": "vqe", "call": "adjoint", "n": 16, "batch": 4096, "layers": 10,
         "terms": 200},
        # VQE: energies only (gradient-free optimisers, evaluation)
        {"name": "vqe_n16_b2048_energy", "family": "vqe", "call": "expectation", "n": 16, "batch": 2048, "layers": 10,
         "terms": 200},
        # energies estimated from measurement shots; an odd size
        {"name": "vqe_n15_b701_shots", "family": "vqe", "call": "sampled", "n": 15, "batch": 701, "layers": 6,
         "terms": 120, "shots": 1000},
        # noisy training step: every circuit ten trajectories; an odd size
        {"name": "vqe_n13_b37x10_noisy", "family": "vqe", "call": "noisy", "n": 13, "batch": 370, "layers": 5,
         "terms": 60, "repeats": 10},
        # a data set of different circuits and qubit counts, default options
        {"name": "ragged_n13_b45_adjoint", "family": "ragged", "call": "adjoint", "n": 13, "batch": 45, "gates": 48,
         "symbols": 12},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A further case: family, call, qubits, depth and batch over the ranges
    the listed cases stand for, at most the largest listed one's work."""
    most = {c["name"]: work(c)["flops"] for c in listed()}
    most = {"grid": most["grid_n30_amplitudes"], "other": most["vqe_n16_b4096_adjoint"]}
    while True:
        fam = rng.choice(("hea", "qnn", "qaoa", "grid", "vqe", "vqe", "ragged"))
        c = {"family": fam}
        if fam == "hea":
            c.update(call=rng.choice(("adjoint", "expectation", "param_shift")), n=rng.randint(3, 9),
                     batch=_log(rng, 8, 1024), layers=rng.randint(1, 4))
        elif fam == "qnn":
            c.update(call=rng.choice(("adjoint", "expectation", "param_shift")), n=rng.randint(6, 13),
                     layers=rng.randint(1, 6))
            c["batch"] = _log(rng, 32, 256 if c["call"] == "param_shift" else 1024)
        elif fam == "qaoa":
            c.update(call=rng.choice(("expectation", "adjoint", "param_shift")), n=2 * rng.randint(5, 11),
                     layers=rng.randint(1, 5))
            c["batch"] = _log(rng, 8, 256 if c["call"] != "param_shift" else 24)
        elif fam == "grid":
            rows, cols = rng.choice(((3, 4), (3, 5), (4, 4), (3, 6), (4, 5), (3, 7), (4, 6), (5, 5), (4, 7), (5, 6)))
            n = rows * cols
            c.update(call="samples", n=n, rows=rows, depth=rng.randint(8, 20), batch=1,
                     shots=0 if n > 25 else _log(rng, 1000, 200000), bitstrings=_log(rng, 100, 4096))
        elif fam == "vqe":
            c.update(call=rng.choice(("adjoint", "expectation", "sampled", "noisy")), n=rng.randint(9, 19),
                     layers=rng.randint(2, 10), terms=_log(rng, 10, 200))
            c["batch"] = _log(rng, 16, 4096)
            if c["call"] == "sampled":
                c["shots"] = _log(rng, 100, 4000)
            if c["call"] == "noisy":
                c["repeats"] = rng.randint(3, 12)
                c["batch"] = c["repeats"] * max(2, c["batch"] // (2 * c["repeats"]))
        else:
            c.update(call=rng.choice(("adjoint", "expectation", "state")), n=rng.randint(6, 15),
                     batch=_log(rng, 8, 96), gates=rng.randint(20, 60), symbols=rng.randint(4, 16))
        # noisy circuits cost several times their noiseless work
        states = (c["batch"] << c["n"]) * (8 if c["call"] == "noisy" else 1)
        if states <= 1 << 30 and work(c)["flops"] <= most.get(fam, most["other"]):
            return c


# ----------------------------------------------------------------- circuits
# A gate is (name, qubits, param); param is None, a number, ("s", symbol,
# scale) or ("row", j): the j-th of the row's own constants.

def _regular3(n):
    """A random 3-regular graph, the same for every call with this n."""
    r = random.Random(3000 + n)
    while True:
        half = [q for q in range(n) for _ in range(3)]
        r.shuffle(half)
        edges = {(min(a, b), max(a, b)) for a, b in zip(half[::2], half[1::2]) if a != b}
        if 2 * len(edges) == 3 * n:
            return sorted(edges)


def _gates(case):
    """(gates, symbols) of a family whose rows share one structure."""
    fam, n, L = case["family"], case["n"], case.get("layers", 0)
    g = []
    if fam == "hea":
        for l in range(L):
            for q in range(n):
                g += [(p, (q,), ("s", (l * n + q) * 3 + a, 1.0)) for a, p in enumerate(("RX", "RY", "RZ"))]
            g += [("CZ", (q, q + 1), None) for q in range(n - 1)]
        return g, 3 * n * L
    if fam == "qnn":
        d = n - 1
        g += [("RX", (i,), ("row", i)) for i in range(d)]
        for l in range(L):
            g += [("ZZPOW", (i, d), ("s", 2 * l * d + i, 1.0)) for i in range(d)]
            g += [("XXPOW", (i, d), ("s", (2 * l + 1) * d + i, 1.0)) for i in range(d)]
        return g, 2 * d * L
    if fam == "qaoa":
        g += [("H", (q,), None) for q in range(n)]
        for l in range(L):
            g += [("RZZ", e, ("s", l, 1.0)) for e in _regular3(n)]
            g += [("RX", (q,), ("s", L + l, 1.0)) for q in range(n)]
        return g, 2 * L
    if fam == "grid":
        rows, cols = case["rows"], n // case["rows"]
        pat = [[(cols * r + c, cols * r + c + 1) for r in range(rows) for c in range(k, cols - 1, 2)] for k in (0, 1)]
        pat += [[(cols * r + c, cols * (r + 1) + c) for r in range(k, rows - 1, 2) for c in range(cols)] for k in (0, 1)]
        r = random.Random(4000 + n)
        last = [None] * n
        for j in range(case["depth"]):
            for q in range(n):
                last[q] = r.choice([x for x in ("SQRTX", "SQRTY", "SQRTW") if x != last[q]])
                g.append((last[q], (q,), None))
            g += [("FSIM", e, None) for e in pat[j % 4]]
        return g, 0
    # vqe
    for l in range(L):
        for q in range(n):
            g.append(("RY", (q,), ("s", 2 * (l * n + q), 1.0)))
            g.append(("RZ", (q,), ("s", 2 * (l * n + q) + 1, 1.0)))
        g += [("CNOT", (q, (q + 1) % n), None) for q in range(n)]
    if case["call"] == "noisy":  # a depolarizing channel after every gate on each of its qubits
        g = [x for a in g for x in [a] + [("DEPOL", (q,), None) for q in a[1]]]
    return g, 2 * n * L


P_NOISE = 0.01


def _terms(case):
    """The family's observable: [(coefficient, [(qubit, letter), ...]), ...]."""
    fam, n = case["family"], case["n"]
    if fam == "hea":
        return [(1.0, [(q, "Z")]) for q in range(n)]
    if fam == "qnn":
        return [(1.0, [(n - 1, "Z")])]
    if fam == "qaoa":
        e = _regular3(n)
        return [(0.5 * len(e), [])] + [(-0.5, [(a, "Z"), (b, "Z")]) for a, b in e]
    r = random.Random(5000 + n)
    seen, out = set(), []
    while len(out) < case["terms"]:
        f = tuple((q, r.choice("XYZ")) for q in sorted(r.sample(range(n), r.randint(1, 4))))
        if f not in seen:
            seen.add(f)
            out.append((r.gauss(0.0, 1.0), list(f)))
    return out


ONE = ("H", "X", "RX", "RY", "RZ", "XPOW", "YPOW", "ZPOW", "SQRTX")
TWO = ("CZ", "CNOT", "XXPOW", "YYPOW", "ZZPOW", "RZZ", "SWAP")
WITH_PARAM = {"RX", "RY", "RZ", "XPOW", "YPOW", "ZPOW", "XXPOW", "YYPOW", "ZZPOW", "RZZ"}


def _ragged(case):
    """Per row (qubits, gates, [two observables])."""
    r = random.Random(6000 + case["n"] * 1000 + case["batch"])
    rows = []
    for b in range(case["batch"]):
        n = case["n"] if b == 0 else r.randint(2, case["n"])
        g = []
        for _ in range(case["gates"]):
            name = r.choice(ONE + TWO)
            qs = tuple(r.sample(range(n), 2 if name in TWO else 1))
            p = None
            if name in WITH_PARAM:
                p = ("s", r.randrange(case["symbols"]), r.uniform(-2, 2)) if r.random() < 0.7 else r.uniform(-3, 3)
            g.append((name, qs, p))
        obs = [[(r.gauss(0, 1), [(q, r.choice("XYZ")) for q in sorted(r.sample(range(n), r.randint(1, min(n, 3))))])
                for _ in range(4)] for _ in range(2)]
        rows.append((n, g, obs))
    return rows


def _circuit(n, gates, row=None):
    c = Circuit(n)
    for name, qs, p in gates:
        if name == "DEPOL":
            c.depolarize(qs[0], P_NOISE)
        elif name == "FSIM":
            c.add(name, qs, [const(math.pi / 2), const(math.pi / 6)])
        elif p is None:
            c.add(name, qs)
        elif isinstance(p, tuple):
            c.add(name, qs, [sym(p[1], p[2]) if p[0] == "s" else const(float(row[p[1]]))])
        else:
            c.add(name, qs, [const(p)])
    return c


def _inputs(case, seed):
    """The seed's numbers, on the host: symbol values, the rows' own
    constants, upstream gradients, bitstrings, stream seeds."""
    rng = np.random.Generator(np.random.PCG64(seed))
    fam, B, n = case["family"], case["batch"], case["n"]
    S = case["symbols"] if fam == "ragged" else _gates(case)[1]
    R = case.get("repeats", 1)
    if fam == "qnn":  # one set of weights, a batch of encoded inputs
        theta = np.repeat(rng.uniform(0, 2 * math.pi, (1, S)), B, axis=0)
    else:
        theta = np.repeat(rng.uniform(0, math.pi if fam == "qaoa" else 2 * math.pi, (B // R, S)), R, axis=0)
    K = 2 if fam == "ragged" else 1
    return {
        "theta": theta.astype(np.float32),
        "rows": math.pi * rng.integers(0, 2, (B, max(n - 1, 1))),
        "upstream": rng.standard_normal((B, K)).astype(np.float32),
        "bits": rng.integers(0, 1 << n, (B, case.get("bitstrings", 1)), dtype=np.int64),
        "seed": int(rng.integers(1, 1 << 62)),
    }


def prepare(case, seed):
    x = _inputs(case, seed)
    B, n = case["batch"], case["n"]
    obs = None
    if case["family"] == "ragged":
        rows = _ragged(case)
        prog = tq.Program(program_blob([_circuit(m, g) for m, g, _ in rows], case["symbols"]))
        obs = tq.Observables(observable_blob([o for _, _, o in rows]))
    else:
        gates, S = _gates(case)
        if case["family"] == "qnn":
            circuits = [_circuit(n, gates, x["rows"][b]) for b in range(B)]
        else:
            circuits = [_circuit(n, gates)] * B
        prog = tq.Program(program_blob(circuits, S), specialize=True)
        if case["call"] != "samples":
            obs = tq.Observables(observable_blob([[_terms(case)]] * B))
    dev = {k: torch.from_numpy(x[k]).cuda() for k in ("theta", "upstream", "bits")}
    return dict(dev, case=case, prog=prog, obs=obs, seed=x["seed"])


def run(s):
    c, prog, obs, theta = s["case"], s["prog"], s["obs"], s["theta"]
    call = c["call"]
    if call in ("adjoint", "noisy"):
        if call == "noisy":
            tq.set_noise_seed(prog, s["seed"])
        e = torch.empty((c["batch"], obs.K), dtype=torch.float32, device="cuda")
        g = tq.adjoint_grad(prog, theta, obs, s["upstream"], expectations=e)
        if call == "noisy":  # a circuit's outputs are the means over its trajectories
            e, g = tq.row_mean(e, c["repeats"]), tq.row_mean(g, c["repeats"])
        return {"expectations": e, "grad": g}
    if call == "expectation":
        return {"expectations": tq.expectation(prog, theta, obs)}
    if call == "param_shift":
        return {"grad": tq.param_shift_grad(prog, theta, obs, s["upstream"])}
    if call == "sampled":
        t = torch.empty((c["batch"], c["terms"]), dtype=torch.float32, device="cuda")
        e = tq.sampled_expectation(prog, theta, obs, c["shots"], s["seed"], term_out=t)
        return {"estimates": e, "terms": t}
    if call == "state":
        return {"states": tq.simulate_state(prog, theta)}
    bits, amps = tq.sample_with_amplitudes(prog, None, c["shots"], s["seed"], s["bits"])
    return {"samples": bits, "amplitudes": amps} if c["shots"] else {"amplitudes": amps}


# --------------------------------------------------------------------- work
# Arithmetic per amplitude: a rotation or square root 6 flops, a diagonal
# phase 3, permutations none, the Hamiltonian 4 per string; the adjoint walks
# psi and phi back (twice the forward work) with 4 per gradient.  Bytes: the
# inputs and outputs, and for states larger than a compute unit's 160 KB of
# local memory one write and one read of every state.
FLOPS = {"CZ": 1, "CNOT": 0, "X": 0, "SWAP": 0, "RZ": 3, "ZPOW": 3, "ZZPOW": 3, "RZZ": 3, "FSIM": 1.5, "DEPOL": 0}


def work(case):
    B, call, n = case["batch"], case["call"], case["n"]
    if case["family"] == "ragged":
        rows = [(m, g, sum(len(t) for t in o)) for m, g, o in _ragged(case)]
        S, K = case["symbols"], 2
    else:
        g, S = _gates(case)
        nt = len(_terms(case)) if call != "samples" else 0
        rows, K = [(n, g, nt)], 1
    mult = B / len(rows)
    if call == "param_shift":
        mult *= 2 * sum(isinstance(p, tuple) and p[0] == "s" for _, _, p in rows[0][1])
    flops = state = 0.0
    for m, g, nt in rows:
        gate = sum(FLOPS.get(name, 6) for name, _, _ in g)
        per = gate + (0 if call in ("state", "samples") else 4 * nt)
        if call in ("adjoint", "noisy"):
            per += 2 * gate + 4 * sum(isinstance(p, tuple) and p[0] == "s" for _, _, p in g)
        flops += mult * per * 2.0 ** m
        if 8 << m > 160 * 1024:
            state += mult * 16.0 * 2.0 ** m
    io = 4.0 * B * (S + K)
    if call in ("adjoint", "noisy", "param_shift"):
        io += 4.0 * B * (S + K)
    if call == "sampled":
        io += 4.0 * B * case["terms"]
    if call == "samples":
        io += 16.0 * case["bitstrings"] + 8.0 * case["shots"]
    if call == "state":
        io += 8.0 * B * 2.0 ** n
    return {"bytes": io + state, "flops": flops}


# complex64 states, fp64 arithmetic: the rounding of stored amplitudes is what
# two correct implementations differ by.  Generated kernels against the
# table-driven ones without fusion: gradients and amplitudes up to 4.8e-7
# (largest single value 7.6e-6), 0.1% of the samples of 24 qubits.
def tolerance(case):
    if case["call"] == "sampled":  # a rounding of a term's value can flip a shot
        return {"rel": 2e-4, "max": 2e-2}
    if case["call"] == "samples":  # a neighbouring bitstring, where the cumulative sum moved
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.006}
    return {"rel": 2e-6, "max": 3e-5}


# -------------------------------------------------------------------- exact
# complex128 states [rows, 2^n] in plain torch.  Qubit q is bit n-1-q.  A gate
# exp(-i a P) is cos a - i sin a P; power gates G^t = e^{i pi t/2} exp(-i pi t/2 G).

ROT = {"RX": "X", "RY": "Y", "RZ": "Z", "RZZ": "ZZ"}
POW = {"XPOW": "X", "YPOW": "Y", "ZPOW": "Z", "XXPOW": "XX", "YYPOW": "YY", "ZZPOW": "ZZ", "SQRTX": "X"}


def _split(psi, n, qubits):
    """psi as [rows, ., 2, ., 2, ...], the size-2 axes at 2, 4, ... in ascending qubit order."""
    shape, at = [psi.shape[0]], 0
    for q in sorted(qubits):
        shape += [1 << (q - at), 2]
        at = q + 1
    return psi.reshape(shape + [1 << (n - at)])


def _pauli(psi, n, factors):
    """P psi for P = [(qubit, letter), ...]."""
    if not factors:
        return psi.clone()
    fs = sorted(factors)
    v = _split(psi, n, [q for q, _ in fs])
    flips = [2 + 2 * i for i, (_, p) in enumerate(fs) if p in "XY"]
    out = v.flip(flips) if flips else v
    w = torch.ones([1] * v.dim(), dtype=psi.dtype, device=psi.device)
    for i, (_, p) in enumerate(fs):
        if p != "X":
            shape = [1] * v.dim()
            shape[2 + 2 * i] = 2
            w = w * torch.tensor({"Y": [-1j, 1j], "Z": [1, -1]}[p], dtype=psi.dtype, device=psi.device).reshape(shape)
    return (out * w).reshape(psi.shape) if w.numel() > 1 else out.reshape(psi.shape)


def _dot(a, b):
    return (a.conj() * b).sum(1)


class _Exact:
    def __init__(self, n, gates, theta, rows, noise_seed=0, row0=0):
        self.n, self.gates, self.theta, self.rows = n, gates, theta, rows
        self.noise_seed, self.row0, self.B = noise_seed, row0, theta.shape[0]

    def eta(self, p):
        """The parameter's value per row, [rows, 1], in fp64."""
        if isinstance(p, tuple):
            return p[2] * self.theta[:, p[1]:p[1] + 1] if p[0] == "s" else self.rows[:, p[1]:p[1] + 1]
        return torch.full((self.B, 1), float(p), dtype=torch.float64, device="cuda")

    def angle(self, gate):
        """(letters, a, da/deta, global phase) of a gate exp(i phase) exp(-i a P)."""
        name, qs, p = gate
        if name in ROT:
            return ROT[name], 0.5 * self.eta(p), 0.5 * (p[2] if isinstance(p, tuple) and p[0] == "s" else 1.0), None
        if name in POW:
            a = 0.5 * math.pi * self.eta(0.5 if p is None else p)
            return POW[name], a, 0.5 * math.pi * (p[2] if isinstance(p, tuple) and p[0] == "s" else 1.0), a
        return None

    def picks(self, k):
        """The Paulis channel k drew in the rows (0 = none, 1 X, 2 Y, 3 Z)."""
        b = np.arange(self.row0, self.row0 + self.B, dtype=np.uint64)
        z = np.uint64(self.noise_seed) + ((b << np.uint64(32) | np.uint64(k)) + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        r, p = ((z ^ (z >> np.uint64(31))) >> np.uint64(11)) * 2.0 ** -53, P_NOISE / 3.0
        return np.where(r < p, 1, np.where(r < p + p, 2, np.where(r < p + p + p, 3, 0)))

    def apply(self, psi, gate, chan, inverse=False):
        name, qs, _ = gate
        n = self.n
        x = self.angle(gate)
        if x is not None:
            letters, a, _, phase = x
            if inverse:
                a, phase = -a, None if phase is None else -phase
            out = torch.cos(a) * psi - 1j * torch.sin(a) * _pauli(psi, n, list(zip(qs, letters)))
            return out if phase is None else torch.exp(1j * phase) * out
        if name == "DEPOL":
            pick = self.picks(chan)
            for k in (1, 2, 3):
                idx = np.nonzero(pick == k)[0]
                if len(idx):
                    i = torch.from_numpy(idx).cuda()
                    psi[i] = _pauli(psi[i], n, [(qs[0], "?XYZ"[k])])
            return psi
        v = _split(psi, n, qs)
        if name == "H":
            a0, a1 = v[:, :, 0], v[:, :, 1]
            return (math.sqrt(0.5) * torch.stack([a0 + a1, a0 - a1], dim=2)).reshape(psi.shape)
        if name == "X":
            return _pauli(psi, n, [(qs[0], "X")])
        out = v.clone()
        lo = qs[0] < qs[1]  # axis 2 is the lower qubit
        at = (lambda a, b: (slice(None), slice(None), a if lo else b, slice(None), b if lo else a))
        if name == "CZ":
            out[at(1, 1)] *= -1
        elif name == "CNOT":
            out[at(1, 0)], out[at(1, 1)] = v[at(1, 1)], v[at(1, 0)]
        else:  # SWAP
            out[at(1, 0)], out[at(0, 1)] = v[at(0, 1)], v[at(1, 0)]
        return out.reshape(psi.shape)

    def forward(self):
        psi = torch.zeros((self.B, 1 << self.n), dtype=torch.complex128, device="cuda")
        psi[:, 0] = 1
        chan = 0
        for g in self.gates:
            psi = self.apply(psi, g, chan)
            chan += g[0] == "DEPOL"
        return psi

    def term_values(self, psi, terms):
        return torch.stack([_dot(psi, _pauli(psi, self.n, f)).real for _, f in terms], dim=1)

    def grad(self, psi, sums, upstream, S):
        """Adjoint gradients of sum_k upstream_k <h_k> and the expectations."""
        phi, e = torch.zeros_like(psi), []
        for k, terms in enumerate(sums):
            h = torch.zeros_like(psi)
            for c, f in terms:
                h += c * _pauli(psi, self.n, f)
            e.append(_dot(psi, h).real)
            phi += upstream[:, k:k + 1] * h
        del h
        out = torch.zeros((self.B, S), dtype=torch.float64, device="cuda")
        chan = sum(g[0] == "DEPOL" for g in self.gates)
        for g in reversed(self.gates):
            chan -= g[0] == "DEPOL"
            if isinstance(g[2], tuple) and g[2][0] == "s":  # Re(-i z) = Im z
                letters, _, da, _ = self.angle(g)
                out[:, g[2][1]] += 2 * da * _dot(phi, _pauli(psi, self.n, list(zip(g[1], letters)))).imag
            psi = self.apply(psi, g, chan, True)
            phi = self.apply(phi, g, chan, True)
        return torch.stack(e, dim=1), out


def _grid_state(n, gates):
    """The state of a grid circuit: its one-qubit layers five qubits at a time, as 32 x 32 matrices."""
    r = math.sqrt(0.5)
    root = {"SQRTX": [[r, -1j * r], [-1j * r, r]], "SQRTY": [[r, -r], [r, r]],
            "SQRTW": [[r, complex(-0.5, -0.5)], [complex(0.5, -0.5), r]]}
    root = {k: complex(r, r) * torch.tensor(m, dtype=torch.complex128) for k, m in root.items()}
    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[0] = 1
    at = 0
    while at < len(gates):
        name, qs, _ = gates[at]
        if name == "FSIM":  # (pi/2, pi/6) on ascending qubits
            v = _split(psi.reshape(1, -1), n, qs)
            x = v[:, :, 0, :, 1].clone()
            v[:, :, 0, :, 1] = -1j * v[:, :, 1, :, 0]
            v[:, :, 1, :, 0] = -1j * x
            v[:, :, 1, :, 1] *= complex(math.cos(math.pi / 6), -math.sin(math.pi / 6))
            at += 1
            continue
        layer = [root[g[0]] for g in gates[at:at + n]]  # qubits 0 .. n-1 in order
        for q in range(0, n, 5):
            k = layer[q]
            for m in layer[q + 1:q + 5]:
                k = torch.kron(k, m)
            v = psi.reshape(1 << q, k.shape[0], -1)
            psi = torch.matmul(k.cuda(), v).reshape(-1)
            del v
        at += n
    return psi


def exact(case, seed):
    x = _inputs(case, seed)
    f64 = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float64)).cuda()  # noqa: E731
    theta, upstream, own = f64(x["theta"]), f64(x["upstream"]), f64(x["rows"])
    B, n, call = case["batch"], case["n"], case["call"]
    if call == "samples":
        amps = _grid_state(n, _gates(case)[0])[torch.from_numpy(x["bits"][0]).cuda()].reshape(1, -1)
        return {"samples": None, "amplitudes": amps} if case["shots"] else {"amplitudes": amps}
    if case["family"] == "ragged":
        parts = []
        for b, (m, g, obs) in enumerate(_ragged(case)):
            parts.append((b, b + 1, m, g, obs))
    else:
        gates, _ = _gates(case)
        sums = [_terms(case)]
        step = max(1, (1 << 23) >> n)  # 128 MiB of amplitudes at a time
        parts = [(b, min(B, b + step), n, gates, sums) for b in range(0, B, step)]
    got = []
    for b0, b1, m, g, sums in parts:
        s = _Exact(m, g, theta[b0:b1], own[b0:b1], x["seed"], b0)
        psi = s.forward()
        if call == "state":
            full = torch.zeros((b1 - b0, 1 << n), dtype=torch.complex128, device="cuda")
            full[:, :1 << m] = psi
            got.append((full,))
        elif call == "sampled":
            got.append((s.term_values(psi, sums[0]),))
        elif call == "expectation":
            got.append((torch.stack([s.term_values(psi, t) @ f64([c for c, _ in t]) for t in sums], dim=1),))
        else:
            got.append(s.grad(psi, sums, upstream[b0:b1], theta.shape[1]))
    out = [torch.cat(v) for v in zip(*got)]
    if call == "noisy":
        out = [v.reshape(B // case["repeats"], case["repeats"], -1).mean(1) for v in out]
    if call in ("adjoint", "noisy"):
        return {"expectations": out[0], "grad": out[1]}
    if call == "param_shift":
        return {"grad": out[1]}
    if call == "sampled":
        return {"estimates": None, "terms": out[0]}
    return {"states" if call == "state" else "expectations": out[0]}

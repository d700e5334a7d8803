"""phi = H psi of the generated gradient passes: Hamiltonians whose terms share
X masks and differ in Z masks on every part of the index (register, thread and
tile bits), from one term per mask to the diagonals of all pairs, with real and
imaginary terms, against the oracle's gradient and expectation."""
import itertools

import numpy as np
import pytest

from gpu_util import compare, dev, gpu_outputs, oracle_outputs
from paper_2003_02989_amd import tq
from paper_2003_02989_amd import workloads as wl
from paper_2003_02989_amd.circuits import Circuit, sym

pytestmark = pytest.mark.gpu


def terms(rng, n, masks, per_mask):
    out = [(0.3, [])]
    for m in range(masks):
        # (four X positions for the largest groups: no three of them fix whether a term is real)
        weight = 4 if per_mask > 100 else int(rng.integers(1, 4)) if m else 0
        xs = set() if m == 0 else set(int(q) for q in rng.choice(n, weight, replace=False))
        for _ in range(per_mask):
            p = []
            for q in range(n):
                z = rng.random() < 0.3
                if q in xs:
                    p.append((q, "Y" if z else "X"))
                elif z:
                    p.append((q, "Z"))
            # the oracle's tolerances hold for observables of norm about 1
            out.append((float(rng.normal()) / (masks * per_mask) ** 0.5, p))
    if masks > 3:
        out += [(0.05, [(i, "Z"), (j, "Z")]) for i in range(n) for j in range(i)]
    return out


def z_patterns(ts, n):
    """The fewest distinct Z patterns that the terms of the last X mask, real and
    imaginary ones apart, have on any three qubits."""
    xs = frozenset(q for q, p in ts[-1][1] if p != "Z")
    group = [(sum(p == "Y" for _, p in f) % 2, {q for q, p in f if p != "X"}) for _, f in ts
             if frozenset(q for q, p in f if p != "Z") == xs]
    return min(len({tuple(q in z for q in bits) for im, z in group if im == part})
               for part in (0, 1) for bits in itertools.combinations(range(n), 3))


@pytest.mark.parametrize("n", [13, 14, 15])
@pytest.mark.parametrize("masks,per_mask", [(1, 1), (2, 1), (2, 4), (3, 40), (6, 9), (2, 150)])
def test_gradient_of_term_groups(n, masks, per_mask):
    rng = np.random.default_rng(1000 * n + 10 * masks + per_mask)
    c = Circuit(n)
    for q in range(n):
        c.add("RY", q, [sym(q % 3, 0.8, 0.1 * q)])
    for q in range(n - 1):
        c.add("CNOT", (q, q + 1))
    for q in range(n):
        c.add("RX", q, [sym((q + 1) % 3, -0.5, 0.2)])
    w = wl.Workload("groups", [c, c], 3, rng.normal(size=(2, 3)).astype(np.float32),
                    [[terms(rng, n, masks, per_mask)]] * 2, rng.normal(size=(2, 1)).astype(np.float32))
    if per_mask == 150:  # more than four masks whichever bits are the registers': summed by butterflies
        assert z_patterns(w.observables[0][0], n) > 4
    compare(gpu_outputs(w, want=("exp", "grad"), specialize=True), oracle_outputs(w, want=("exp", "grad")))
    p, o = tq.Program(w.program_blob(), specialize=True), tq.Observables(w.observable_blob())
    tq.adjoint_grad(p, dev(w.theta), o, dev(w.upstream))
    # the generated passes ran, and hold every term but the constant
    assert sum(tq.describe(p)["groups"][0]["obs"]["phi_passes"]) >= len(w.observables[0][0]) - 1

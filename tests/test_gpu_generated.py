"""Generated kernels (specialize) against the oracle on circuits that mix the
ops their stages treat specially: X and CNOT gates turned into index maps of a
stage's loads and stores (controls inside and outside the stage and the tile,
chains, plain X, targets and controls touched before and after) and Z-type
gradients taken together, among rotations and diagonal gates that keep them
from moving; and rotations applied as shears, at the angles where a shear
changes sign or its entries are extreme.  Sizes: resident circuits, states
of one tile and of several."""
import numpy as np
import pytest
import torch

from gpu_util import compare, dev, gpu_outputs, oracle_outputs, say
from paper_2003_02989_amd import tq
from paper_2003_02989_amd import workloads as wl
from paper_2003_02989_amd.circuits import Circuit, sym

pytestmark = pytest.mark.gpu

POOLS = {
    "x": ["X", "CNOT", "CNOT", "CNOT", "RY", "RZ", "RZ", "CZPOW"],
    "mixed": ["X", "CNOT", "CNOT", "RX", "RY", "RZ", "ZZPOW", "RZZ", "XXPOW", "H", "SWAP", "CZ", "CNOTPOW"],
}


def batch(pool, n, gates, seed, B=3):
    rng = wl.rng_for(seed)
    c = wl.random_circuit(rng, n, gates, 7, ops=POOLS[pool])
    obs = wl.random_observables(rng, n, 1, max_terms=8, max_weight=min(n, 4))
    theta = rng.uniform(-3.2, 3.2, size=(B, 7)).astype("float32")
    up = rng.standard_normal((B, 1)).astype("float32")
    return wl.Workload(f"{pool}_n{n}", [c] * B, 7, theta, [obs] * B, up)


@pytest.mark.parametrize("pool", sorted(POOLS))
@pytest.mark.parametrize("n,gates", [(3, 40), (6, 90), (10, 120), (13, 160), (15, 220)])
def test_generated_against_oracle(pool, n, gates):
    w = batch(pool, n, gates, 9100 + n)
    say(w.name)
    compare(gpu_outputs(w, specialize=True), oracle_outputs(w))


@pytest.mark.parametrize("n", [5, 14])
def test_cnot_chains(n):
    # a ring both ways round, X between, no op in some stages but permutations
    c = Circuit(n)
    for q in range(n):
        c.add("RY", q, [sym(q % 4, 0.7 + 0.1 * q, 0.2)])
    for q in range(n):
        c.add("CNOT", (q, (q + 1) % n))
    for q in range(0, n, 3):
        c.add("X", q)
    for q in reversed(range(n)):
        c.add("CNOT", ((q + 1) % n, q))
    for q in range(n):
        c.add("RZ", q, [sym((q + 1) % 4, 1.0 - 0.05 * q)])
        c.add("CNOT", (q, (q + 2) % n))
    rng = wl.rng_for(77)
    obs = wl.random_observables(rng, n, 1, max_terms=6, max_weight=3)
    theta = rng.uniform(-3, 3, size=(2, 4)).astype("float32")
    w = wl.Workload(f"chain_n{n}", [c] * 2, 4, theta, [obs] * 2, rng.standard_normal((2, 1)).astype("float32"))
    compare(gpu_outputs(w, specialize=True), oracle_outputs(w))


@pytest.mark.parametrize("n", [4, 13, 14])
def test_rotation_shears_at_special_angles(n):
    # multiples of pi/2 and their neighbours, many turns, tiny angles: states
    # compare with their phase (a sign left out by a shear joins the row's
    # phase), and fused rotations about one axis take the sum of their angles
    pi = np.pi
    angles = [0.0, pi / 2, pi, -pi, 3 * pi / 2, 2 * pi, -2 * pi, 3 * pi, 4 * pi, 1e-7, pi - 1e-6, pi + 1e-6, 41.3, -57.9]
    rng = wl.rng_for(31 + n)
    c = Circuit(n)
    for q in range(n):
        c.add("H", q)
        c.add("CZ", (q, (q + 1) % n))
    for j, op in enumerate(["RY", "RX", "YPOW", "XPOW"] * 2):
        for q in range(n):
            c.add(op, q, [sym((j + q) % 5, 1.0 if op[0] == "R" else 1.0 / pi)])
            if q % 3 == 0:  # a second rotation about the same axis fuses
                c.add(op, q, [sym((j + q + 1) % 5, -0.5)])
        c.add("XXPOW" if j % 2 else "YYPOW", (j % n, (j + 2) % n), [sym(j % 5, 1.0 / pi)])
        c.add("CNOT", (j % n, (j + 1) % n))
    theta = rng.choice(angles, size=(6, 5)).astype("float32")
    obs = wl.random_observables(rng, n, 1, max_terms=6, max_weight=3)
    w = wl.Workload(f"angles_n{n}", [c] * 6, 5, theta, [obs] * 6, np.ones((6, 1), "float32"))
    compare(gpu_outputs(w, specialize=True), oracle_outputs(w))


@pytest.mark.parametrize("n", [1, 2, 6, 7, 9, 10, 11, 12])
def test_resident_sizes(n):
    # the product state by thread and register bits: fewer amplitudes than
    # threads, one each, and every count of shared bits; first gates dense
    rng = wl.rng_for(9500 + n)
    c = Circuit(n)
    for q in range(n):
        c.add("RX", q, [sym(q % 3, 0.5, 0.1 * q)]).add("RZ", q, [sym((q + 1) % 3, 1.0, 0.2)]).add("RY", q, [sym(q % 3)])
    for q in range(n - 1):
        c.add("CZ", (q, q + 1)).add("RY", q, [sym(q % 3, -0.7)])
    obs = wl.random_observables(rng, n, 2, max_terms=5, max_weight=min(n, 3))
    theta = rng.uniform(-3, 3, size=(3, 3)).astype("float32")
    w = wl.Workload(f"resident_n{n}", [c] * 3, 3, theta, [obs] * 3, rng.standard_normal((3, 2)).astype("float32"))
    compare(gpu_outputs(w, specialize=True), oracle_outputs(w))


def test_first_forward_call_inside_a_capture():
    # after a gradient alone nothing forward is loaded: the whole kernel runs
    w = batch("mixed", 7, 60, 9600)
    p, o, th = tq.Program(w.program_blob(), specialize=True), tq.Observables(w.observable_blob()), dev(w.theta)
    tq.adjoint_grad(p, th, o, dev(w.upstream))
    out = torch.empty((w.B, w.K), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tq.expectation(p, th, o, out=out)
    ref = tq.expectation(p, th, o)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert (out - ref).abs().max().item() <= 1e-5

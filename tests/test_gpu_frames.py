"""Pauli frames: noisy circuits of Clifford gates and rotations (channels moved
to the end, angles negated) against the oracle's trajectories, row by row, for
states with their phase, expectations, adjoint and shift-rule gradients, on
the generated and the table-driven kernels; resident circuits, one tile, and
several tiles; uniform rows, per-row constants and several structures."""
import numpy as np
import pytest

from gpu_util import TOL_GRAD, compare, dev, oracle_outputs
from oracle import oracle as orc
from paper_2003_02989_amd import tq
from paper_2003_02989_amd import workloads as wl
from paper_2003_02989_amd.circuits import Circuit, const, sym

pytestmark = pytest.mark.gpu
ROT1, ROT2 = ["RX", "RY", "RZ", "XPOW", "YPOW", "ZPOW"], ["XXPOW", "YYPOW", "ZZPOW", "RZZ"]
FIXED1, FIXED2 = ["H", "X", "Y", "Z", "SQRTX", "SQRTY"], ["CZ", "CNOT", "SWAP"]


def noisy_circuit(rng, n, gates, S, value=0.4):
    """Random Clifford gates and rotations, a channel after most of them."""
    c = Circuit(n)
    for _ in range(gates):
        pool = [ROT1, FIXED1] + ([ROT2, FIXED2] if n > 1 else [])
        name = str(rng.choice(pool[int(rng.integers(len(pool)))]))
        nq = 1 if name in ROT1 + FIXED1 else 2
        qs = tuple(int(q) for q in rng.choice(n, size=nq, replace=False))
        par = []
        if name in ROT1 + ROT2:
            par = [sym(int(rng.integers(S)), float(rng.uniform(-2, 2)), 0.3)] if rng.random() < 0.7 else [const(value)]
        c.add(name, qs, par)
        for q in qs:
            if rng.random() < 0.7:
                c.add("PCHAN", q, [float(p) for p in rng.uniform(0, 0.3, 3)])
    return c


def check(w, noise_seed, shift=False, **opts):
    orc.set_noise_seed(noise_seed)
    orc.set_row_offset(0)
    p = tq.Program(w.program_blob(), **opts)
    tq.set_noise_seed(p, noise_seed)
    o, th = tq.Observables(w.observable_blob()), dev(w.theta)
    out = {"state": tq.simulate_state(p, th).cpu().numpy(), "exp": tq.expectation(p, th, o).cpu().numpy()}
    e = dev(np.zeros((w.B, w.K)))
    out["grad"] = tq.adjoint_grad(p, th, o, dev(w.upstream), expectations=e).cpu().numpy()
    out["grad_exp"] = e.cpu().numpy()
    ref = oracle_outputs(w)
    compare(out, ref)
    if shift:
        g = tq.param_shift_grad(p, th, o, dev(w.upstream)).cpu().numpy()
        assert np.abs(g - ref["grad"]).max() <= TOL_GRAD


def workload(rng, circuits, S, K=2):
    B = len(circuits)
    obs = [wl.random_observables(rng, c.n, K, max_terms=6, max_weight=min(c.n, 4)) for c in circuits]
    if all(c is circuits[0] for c in circuits):
        obs = [obs[0]] * B
    theta = rng.uniform(-3, 3, size=(B, S)).astype("float32")
    return wl.Workload("frames", circuits, S, theta, obs, rng.standard_normal((B, K)).astype("float32"))


@pytest.mark.parametrize("specialize", [False, True])
@pytest.mark.parametrize("n,gates,K", [(1, 12, 1), (3, 40, 2), (7, 80, 1), (12, 90, 1), (13, 110, 1), (14, 120, 2)])
def test_against_oracle(n, gates, K, specialize):
    rng = wl.rng_for(6100 + n)
    c = noisy_circuit(rng, n, gates, 4)
    w = workload(rng, [c] * 5, 4, K)
    for seed in (3, 4):
        check(w, seed, shift=n <= 7 or n == 13, specialize=specialize)


@pytest.mark.parametrize("specialize", [False, True])
def test_many_rotations_and_per_row_constants(specialize):
    # more than 64 frame words per row, rows that differ in their constants
    rng = wl.rng_for(6200)
    base = [noisy_circuit(wl.rng_for(6201), 2, 4200, 3, value=0.1 * b) for b in range(3)]
    w = workload(rng, base, 3)
    assert len(tq.describe(tq.Program(w.program_blob()))["groups"]) == 1
    check(w, 9, specialize=specialize)


@pytest.mark.parametrize("gates", [30, 60, 130, 400, 900, 2000, 2300, 3700])
def test_frame_widths(gates):
    # a frame's words side by side in a wavefront: from 32 channels of two words
    # to one of 64, and in strips; most channels draw a Pauli
    rng = wl.rng_for(6600 + gates)
    c = noisy_circuit(rng, 2, gates, 3)
    for q in (0, 1):
        for _ in range(40):
            c.add("PCHAN", q, [0.3, 0.3, 0.3])
    check(workload(rng, [c] * 3, 3), 11, specialize=gates < 200)


def test_several_structures():
    rng = wl.rng_for(6300)
    w = workload(rng, [noisy_circuit(rng, n, 30, 3) for n in (2, 5, 9, 13)], 3)
    check(w, 21)


def test_gates_without_frames_keep_their_channels():
    rng = wl.rng_for(6400)
    c = noisy_circuit(rng, 5, 40, 3).add("CNOTPOW", (0, 1), [sym(0)]).depolarize(1, 0.4).add("SQRTW", 2)
    check(workload(rng, [c] * 4, 3), 5, specialize=True)

"""The signs that the shears of rotations leave to a row's global phase: states
of generated kernels against the oracle with angles of any size, with rotations
at odd quarter turns in more build tasks than one workgroup builds, and the
builder's matrices against the host's."""
import numpy as np
import pytest

from gpu_util import TOL_AMP, TOL_EXP, gpu_outputs, oracle_outputs
from paper_2003_02989_amd import tq
from paper_2003_02989_amd import workloads as wl
from paper_2003_02989_amd.circuits import Circuit, sym
from test_gpu_builder import check

pytestmark = pytest.mark.gpu
FAR = [1e5, 2.0**39, 2.0**41, 1e15, -1e16, 3e17, -1e20, 1e25, 1e30, 3e38]


def rotations(n, names1, names2):
    """Rotations behind an entangled state, also two about one axis in a row."""
    c = Circuit(n)
    for q in range(n):
        c.add("H", q).add("RZ", q, [0.3 * q])
    for q in range(n - 1):
        c.add("CNOT", (q, q + 1))
    for k, name in enumerate(names1):
        for q in range(n):
            c.add(name, q, [sym(0, 1.0 if (q + k) % 2 else -2.0)])
            if q % 2:
                c.add(name, q, [sym(1, 1.0, 0.0)])
        for q in range(n - 1):
            c.add("CZ", (q, q + 1))
    for k, name in enumerate(names2):
        c.add(name, (k, k + 1), [sym(0, 0.5)]).add("CZ", (k, n - 1))
    return c


def workload(c, theta):
    n, B = c.n, len(theta)
    obs = [[(0.5, [(0, "X")]), (0.5, [(n - 1, "Z")])]]
    return wl.Workload("far", [c] * B, 2, np.asarray(theta, np.float32), [obs] * B, np.ones((B, 1), np.float32))


@pytest.mark.parametrize("specialize", [True, False])
@pytest.mark.parametrize("n", [4, 13])
def test_radians_of_any_size(n, specialize):
    w = workload(rotations(n, ["RX", "RY", "RX"], []), [[v, u] for v, u in zip(FAR, [0.4, -2.0] * 5)] + [[v, -v] for v in FAR])
    got, ref = gpu_outputs(w, want=("state", "exp"), specialize=specialize), oracle_outputs(w, want=("state", "exp"))
    assert np.linalg.norm(got["state"] - ref["state"], axis=1).max() <= TOL_AMP
    assert np.abs(got["exp"] - ref["exp"]).max() <= TOL_EXP


# doubles whose half is within 1e-9 of an odd multiple of pi (convergents of 2^a
# / pi): the rotation is minus the identity, which the angle's nearest multiple
# of pi in fp64 does not tell
ODD = [2.0 * m * 2.0**a for a, m in ((20, 11923407502), (30, 8044219540), (40, 1714902710), (50, 2132823294),
                                     (60, 723010357), (70, 1967564526), (80, 3108327914))]


@pytest.mark.parametrize("n", [4, 13])
@pytest.mark.parametrize("eta", ODD)
def test_odd_multiples_of_pi(n, eta):
    c = Circuit(n)
    for q in range(n):
        c.add("H", q).add("RZ", q, [0.3 * q])
    for q in range(n - 1):
        c.add("CNOT", (q, q + 1))
    for q in range(n):
        c.add(("RX", "RY")[q % 2], q, [sym(0, 1.0, eta if q % 3 else -eta)])
    w = workload(c, [[0.0, 0.0]])
    got, ref = gpu_outputs(w, want=("state", "exp"), specialize=True), oracle_outputs(w, want=("state", "exp"))
    assert np.linalg.norm(got["state"] - ref["state"], axis=1).max() <= TOL_AMP
    assert np.abs(got["exp"] - ref["exp"]).max() <= TOL_EXP


@pytest.mark.parametrize("specialize", [True, False])
@pytest.mark.parametrize("n", [4, 13])
def test_powers_of_any_size(n, specialize):
    # periodic in the exponent up to the state's phase (whose own terms grow
    # with the exponent): the states of the reduced exponents, up to a phase
    far = np.asarray([[s * 2.0**k + 2.0**max(k - 22, -2), 0.25] for k in (3, 12, 21) for s in (1, -1)] +
                     [[s * 2.0**k, 0.25] for k in (30, 53, 62, 63, 64, 70, 126) for s in (1, -1)], np.float32)
    c = rotations(n, ["XPOW", "YPOW", "XPOW"], ["XXPOW", "YYPOW"])
    # (reduced modulo 8: the scales go down to 1/2 and the periods are 2)
    near = np.fmod(far.astype(np.float64), 8.0)
    got, ref = gpu_outputs(workload(c, far), want=("state", "exp"), specialize=specialize), \
        oracle_outputs(workload(c, near), want=("state", "exp"))
    overlap = np.abs(np.sum(ref["state"].conj() * got["state"], axis=1))
    norm = np.linalg.norm(got["state"], axis=1)
    assert np.abs(overlap - 1).max() <= TOL_AMP and np.abs(norm - 1).max() <= TOL_AMP
    assert np.abs(got["exp"] - ref["exp"]).max() <= TOL_EXP


def many_tasks(rng, n, layers):
    c = Circuit(n)
    for _ in range(layers):
        for q in range(n):
            name = str(rng.choice(["XPOW", "YPOW"]))
            for _ in range(2):  # sums of quarters: odd multiples of half a turn among them
                c.add(name, q, [sym(int(rng.integers(2)), float(rng.choice([-1, 1, 3, 5])), float(rng.integers(-2, 3)))])
        for q in range(n - 1):
            c.add("CNOT", (q, q + 1))
    return c


@pytest.mark.parametrize("n", [5, 13])
def test_ties_beyond_one_workgroup(n):
    rng = np.random.default_rng(n)
    c = many_tasks(rng, n, 60)
    w = workload(c, [[0.5, 0.5], [0.25, 0.75], [1.5, -0.5], [0.125, 0.25]])
    d = tq.describe(tq.Program(w.program_blob(), specialize=True))["groups"][0]
    assert sum(t[0] == 0 for t in d["tasks"]) > 256
    got, ref = gpu_outputs(w, want=("state",), specialize=True), oracle_outputs(w, want=("state",))
    assert np.linalg.norm(got["state"] - ref["state"], axis=1).max() <= TOL_AMP


@pytest.mark.parametrize("specialize", [True, False])
def test_matrices_of_odd_turns(specialize):
    # the matrices hold their own signs: the phase beside them takes none up
    w = workload(rotations(4, ["RX", "YPOW"], ["XXPOW"]), [[v, 0.3] for v in (1.0, 3.0, 5.0, 7.0, 9.0)])
    assert check(w, specialize=specialize) < 1e-12

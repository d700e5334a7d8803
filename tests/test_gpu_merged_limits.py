"""Merged launches beside what the groups' own launches need: calls captured
after eager ones of another kind, and the memory a call takes."""
import numpy as np
import pytest
import torch

from gpu_util import TOL_AMP, TOL_EXP, TOL_GRAD, compare, dev, gpu_outputs, oracle_outputs
from paper_2003_02989_amd import tq
from paper_2003_02989_amd import workloads as wl
from paper_2003_02989_amd.circuits import Circuit, sym

pytestmark = pytest.mark.gpu


def mixed(seed, sizes, K, zonly=False):
    rng = wl.rng_for(seed)
    circuits = [wl.random_circuit(rng, n, 40, 3) for n in sizes]
    theta = rng.uniform(-3, 3, size=(len(sizes), 3)).astype("float32")
    obs = [wl.random_observables(rng, n, K, max_terms=6, max_weight=min(n, 3)) for n in sizes]
    if zonly:
        obs = [[[(c, [(q, "Z") for q, _ in f]) for c, f in t] for t in row] for row in obs]
    return wl.Workload("mixed", circuits, 3, theta, obs, rng.standard_normal((len(sizes), K)).astype("float32"))


def replayed(graph, out, eager, th):
    for k in range(3):
        th.mul_(1.0 + 0.1 * k)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        assert np.abs((got - eager()).cpu().numpy()).max() <= TOL_GRAD


def test_diagonal_expectation_captured_after_a_gradient():
    # Z-only observables of larger states keep their own kernel
    w = mixed(11, [13, 13, 2, 14], 2, zonly=True)
    p, o = tq.Program(w.program_blob()), tq.Observables(w.observable_blob())
    th, up = dev(w.theta), dev(w.upstream)
    e = torch.empty((w.B, w.K), dtype=torch.float32, device="cuda")
    tq.adjoint_grad(p, th, o, up)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tq.expectation(p, th, o, out=e)
    graph.replay()
    torch.cuda.synchronize()
    assert np.abs(e.cpu().numpy() - oracle_outputs(w, want=("exp",))["exp"]).max() <= TOL_EXP
    replayed(graph, e, lambda: tq.expectation(p, th, o), th)


def test_states_captured_after_an_expectation():
    w = mixed(13, [13, 5, 2], 1)
    p, o, th = tq.Program(w.program_blob()), tq.Observables(w.observable_blob()), dev(w.theta)
    st = torch.empty((w.B, 2**13), dtype=torch.complex64, device="cuda")
    tq.expectation(p, th, o)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tq.simulate_state(p, th, out=st)
    graph.replay()
    torch.cuda.synchronize()
    assert np.linalg.norm(st.cpu().numpy() - oracle_outputs(w, want=("state",))["state"], axis=1).max() <= TOL_AMP
    replayed(graph, st, lambda: tq.simulate_state(p, th), th)


def test_gradient_of_a_second_observable_set_captured():
    w, wb = mixed(12, [13, 14, 3], 2), mixed(12, [13, 14, 3], 2, zonly=True)
    p, oa, ob = tq.Program(w.program_blob()), tq.Observables(w.observable_blob()), tq.Observables(wb.observable_blob())
    th, up = dev(w.theta), dev(w.upstream)
    g = torch.empty((w.B, 3), dtype=torch.float32, device="cuda")
    tq.adjoint_grad(p, th, oa, up)
    tq.expectation(p, th, ob)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tq.adjoint_grad(p, th, ob, up, grad=g)
    graph.replay()
    torch.cuda.synchronize()
    ref = oracle_outputs(wl.Workload("b", w.circuits, 3, w.theta, wb.observables, w.upstream), want=("grad",))["grad"]
    assert np.abs(g.cpu().numpy() - ref).max() <= TOL_GRAD
    replayed(graph, g, lambda: tq.adjoint_grad(p, th, ob, up), th)


@pytest.mark.parametrize("rows", [4096, 4097])
def test_structures_of_many_rows_beside_small_ones(rows):
    # up to 4096 rows of a structure are merged, more run by themselves
    rng = wl.rng_for(14)
    a, b = wl.random_circuit(rng, 2, 12, 2), wl.random_circuit(rng, 3, 12, 2)
    B = rows + 3
    w = wl.Workload("rows", [b, b] + [a] * rows + [b], 2, rng.uniform(-3, 3, size=(B, 2)).astype("float32"),
                    [[[(0.6, [(0, "X"), (1, "Z")]), (0.2, [(1, "Y")])]]] * B, rng.standard_normal((B, 1)).astype("float32"))
    compare(gpu_outputs(w), oracle_outputs(w))


def test_memory_of_many_small_rows_beside_a_large_one():
    # an expectation takes the rows' states; no table grows with rows x 2^nmax
    n, small = 24, 4000
    big = Circuit(n)
    for q in range(n):
        big.add("RX", q, [sym(0, 0.1 * q)])
    for q in range(n - 1):
        big.add("CNOT", (q, q + 1))
    tiny = Circuit(2).add("RY", 0, [sym(0)]).add("CNOT", (0, 1))
    B = small + 1
    w = wl.Workload("memory", [big] + [tiny] * small, 1, np.linspace(-3, 3, B, dtype=np.float32)[:, None],
                    [[[(1.0, [(0, "Z"), (1, "X")])]]] * B, np.ones((B, 1), np.float32))
    p, o, th = tq.Program(w.program_blob()), tq.Observables(w.observable_blob()), dev(w.theta)
    e = torch.empty((B, 1), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    tq.expectation(p, th, o, out=e)
    torch.cuda.synchronize()
    took = free - torch.cuda.mem_get_info()[0]
    state = 8 * 2**n
    assert took <= state + (48 << 20), took  # matrices, tables and partial sums beside it: some MB


def test_memory_of_many_parameters_on_large_states():
    # the gradient sums of all structures side by side would take 590 MB
    n, G, S = 22, 12, 6000
    sums = 8 * S * 2 ** (n - 12)  # of one structure
    circuits = []
    for k in range(G):
        c = Circuit(n)
        for q in range(n):
            c.add("RY", q, [0.1 + 0.2 * q])
        for i in range(S):
            c.add("RZ", (i + k) % n, [sym(0, 0.001 * (1 + i % 7))])
        circuits.append(c.add("CNOT", (k, k + 1)))
    theta = np.linspace(-1, 1, G, dtype=np.float32)[:, None]
    obs = [[[(0.7, [(0, "X"), (5, "X")]), (0.4, [(k, "Y")])]] for k in range(G)]
    w = wl.Workload("params", circuits, 1, theta, obs, np.ones((G, 1), np.float32))
    p, o, th, up = tq.Program(w.program_blob()), tq.Observables(w.observable_blob()), dev(w.theta), dev(w.upstream)
    g = torch.empty((G, 1), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    tq.adjoint_grad(p, th, o, up, grad=g)
    torch.cuda.synchronize()
    took = free - torch.cuda.mem_get_info()[0] - 2 * 8 * G * 2**n
    # 256 MB, passed by one structure's at most, and the program's own for one structure
    assert took <= (256 << 20) + 2 * sums + (64 << 20), took
    for k in (0, 6, G - 1):
        one = wl.Workload("one", [circuits[k]], 1, theta[k : k + 1], [obs[k]], w.upstream[:1])
        ref = gpu_outputs(one, want=("grad",))["grad"]
        assert np.abs(g[k].cpu().numpy() - ref[0]).max() <= TOL_GRAD

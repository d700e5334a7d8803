"""Whole-state reverse tiles with as many gradient slots as their LDS takes, and
one more (a second pass), and with every kind of op, against the oracle."""
import numpy as np
import pytest

from gpu_util import compare, gpu_outputs, oracle_outputs
from paper_2003_02989_amd import workloads as wl
from test_rev_tile_cpu import ansatz, limit, rev_tile

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("low", [3, 6])
@pytest.mark.parametrize("over", [0, 1])
def test_gradient_at_the_slot_limit(low, over):
    rng = np.random.default_rng(low)
    c = ansatz(limit(13 - low) + over)
    w = wl.Workload("rev", [c] * 3, 7, rng.normal(size=(3, 7)).astype(np.float32),
                    [[[(0.7, [(0, "Z"), (5, "X")]), (0.4, [(12, "Y")])]]] * 3, rng.normal(size=(3, 1)).astype(np.float32))
    compare(gpu_outputs(w, want=("exp", "grad"), specialize=True, low_qubits=low),
            oracle_outputs(w, want=("exp", "grad")))


@pytest.mark.parametrize("rows,t", [(2, 12), (130, 13), (260, 12)])
def test_gradient_of_dense_circuits(rows, t):
    rng = wl.rng_for(13)
    c = wl.random_circuit(rng, 13, 150, 7)
    assert rev_tile(c, rows)[0] == t
    w = wl.Workload("dense", [c] * rows, 7, rng.uniform(-3, 3, size=(rows, 7)).astype(np.float32),
                    [wl.random_observables(rng, 13, 1, max_terms=6, max_weight=3)] * rows,
                    rng.normal(size=(rows, 1)).astype(np.float32))
    compare(gpu_outputs(w, want=("exp", "grad"), specialize=True), oracle_outputs(w, want=("exp", "grad")))

"""Whole-state reverse tiles with as many gradient slots as their LDS takes, and
one more (a second pass), against the oracle."""
import numpy as np
import pytest

from gpu_util import compare, gpu_outputs, oracle_outputs
from paper_2003_02989_amd import workloads as wl
from test_rev_tile_cpu import ansatz, limit

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

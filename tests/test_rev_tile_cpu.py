"""Plans of the whole-state reverse tile (13 qubits, generated kernels): the
pass's LDS -- two states of 2^13 amplitudes, the offset table of 2^h entries
and eight wavefronts' gradient sums -- fits a CU's 160 KB for every low_qubits
the options allow and for slot counts around the limit that follows."""
import numpy as np
import pytest

from paper_2003_02989_amd import tq
from paper_2003_02989_amd import workloads as wl
from paper_2003_02989_amd.circuits import Circuit, sym

CU_LDS = 160 * 1024


def ansatz(slots, n=13):
    """Layers of RY, RZ and a CNOT ring with `slots` symbolic angles in all."""
    c = Circuit(n)
    k = 0
    while k < slots:
        for q in range(n):
            for op in ("RY", "RZ"):
                if k < slots:
                    c.add(op, q, [sym(k % 7, 1.0, 0.01 * k)])
                    k += 1
        for q in range(n):
            c.add("CNOT", (q, (q + 1) % n))
    return c


def plan(slots, low):
    w = wl.Workload("rev", [ansatz(slots)], 7, np.zeros((1, 7), np.float32), [[[(1.0, [(0, "Z")])]]],
                    np.ones((1, 1), np.float32))
    return tq.describe(tq.Program(w.program_blob(), specialize=True, **({"low_qubits": low} if low else {})))["groups"][0]


def limit(h):
    return (CU_LDS - 2 * 8 * 2**13 - 8 * 2**h) // (8 * 8)


@pytest.mark.parametrize("low", [0, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("over", [-60, -1, 0, 1, 60, 500])
def test_whole_state_tile_fits_the_lds(low, over):
    h = 13 - (low or 6)
    slots = limit(h) + over
    g = plan(slots, low)
    got = 0
    for ps in g["rev"]:
        gcount = sum(op["ngrad"] for op in ps["ops"])
        got += gcount
        assert ps["t"] == 13 and ps["h"] == h
        assert 2 * 8 * 2**ps["t"] + 8 * 2**ps["h"] + 8 * 8 * gcount <= CU_LDS
    assert got == slots
    # one pass where one fits
    assert len(g["rev"]) == -(-slots // limit(h))

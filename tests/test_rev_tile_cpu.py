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


def rev_tile(c, rows, **kw):
    w = wl.Workload("rows", [c] * rows, 7, None, None, None)
    rev = tq.describe(tq.Program(w.program_blob(), specialize=True, **kw))["groups"][0]["rev"]
    return rev[0]["t"], len(rev), sum(len(ps["stages"]) for ps in rev)


# rows: up to 128, one round of the chip's 256 CUs, full rounds, a last round mostly empty
ROWS = [1, 128, 129, 256, 257, 352, 448, 512, 600, 1024]


@pytest.mark.parametrize("kind,wholes", [
    ("layers", ROWS),                            # few stages per pass saved
    ("dense", [129, 256, 448, 512, 1024]),       # many
    ("one pass", []),                            # none saved
])
def test_whole_state_tiles_where_they_pay(kind, wholes):
    if kind == "layers":
        c = ansatz(130)
    elif kind == "dense":
        c = wl.random_circuit(wl.rng_for(13), 13, 150, 7)
    else:
        c = Circuit(13)
        for q in range(13):
            c.add("RZ", q, [sym(q % 7)]).add("CZPOW", (q, (q + 1) % 13), [sym((q + 1) % 7)])
    t12, p12, _ = rev_tile(c, 1, max_tile_qubits=13)
    assert t12 == 12
    for rows in ROWS:
        t, passes, stages = rev_tile(c, rows)
        assert t == (13 if rows in wholes else 12), rows
        assert passes == (1 if t == 13 else p12)
    if kind != "one pass":
        _, _, stages = rev_tile(c, 256)
        assert (stages <= 6 * (p12 - 1)) == (kind == "layers") and (stages > 11 * (p12 - 1)) == (kind == "dense")

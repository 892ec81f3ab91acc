"""Dense export of stabilizer states at the edges of its tiles (2^12 indices):
states below, at and above one tile, with no X-type generator (a basis
state), one (GHZ), all of them (every qubit in superposition) and random
ones. Against the oracle up to the global phase: every amplitude is
2^{-r/2} i^e rounded once to FP32, so it agrees within 2^-23 of its
magnitude."""
import numpy as np
import pytest

import oracle
from tests.test_tableau_host import random_clifford

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2609_23664_amd import binding as B
    return B.Ctx(0)


def _circuits(n):
    g = np.random.default_rng(40 + n)
    yield "basis", [("X", (q,), 0.0) for q in range(0, n, 2)]
    yield "ghz", [("H", (n - 1,), 0.0)] + [("CNOT", (q, q - 1), 0.0) for q in range(n - 1, 0, -1)] + [("S", (0,), 0.0)]
    yield "graph", ([("H", (q,), 0.0) for q in range(n)] + [("CZ", (q, (q + 1) % n), 0.0) for q in range(n) if n > 2]
                    + [("SDG", (q,), 0.0) for q in range(0, n, 3)] + [("X", (n // 2,), 0.0)])
    for k in range(3):
        yield f"random{k}", random_clifford(n, g, 12 * n)


@pytest.mark.parametrize("n", [2, 3, 11, 12, 13, 14, 18])
def test_export_tile_edges(ctx, n):
    from paper_2609_23664_amd import binding as B
    st = B.State(ctx, n, 1)
    for name, gates in _circuits(n):
        print("[gpu-case] export", n, name, flush=True)
        tb = B.Tableau(n)
        tb.apply(gates)
        tb.export(st, 0)
        psi = st.host(0).astype(np.complex128)
        ref = oracle.simulate(n, gates)
        k = int(np.argmax(np.abs(ref)))
        assert abs(psi[k]) > 0.0, name
        ref = ref * (psi[k] / abs(psi[k])) / (ref[k] / abs(ref[k]))
        assert np.max(np.abs(psi - ref)) <= 2.0 ** -23 * np.max(np.abs(ref)), name
        tb.free()
    st.free()

"""Measurement masses and decisions at the edges of their kernels: chunks of
256, 512 and 1,024 amplitudes, bins of one chunk up to more than 256 chunks,
1 to 12 joint measurements, single measurements of the lowest and highest
qubit. Random states against the oracle's sequential Born rule; every draw is
at least 1e-3 away from its outcome probability, so the outcomes are exact
and the state agrees within the FP32 bar (1 - F <= 1e-6)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2609_23664_amd import binding as B
    return B.Ctx(0)


def _case(n, qs, seed):
    rng = np.random.default_rng(seed)
    psi = (rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)).astype(np.complex64)
    psi /= np.linalg.norm(psi)
    w = np.abs(psi.astype(np.complex128)) ** 2
    idx = np.arange(1 << n)
    gates = []
    for q in qs:
        one = (idx >> q) & 1 == 1
        p1 = w[one].sum() / w.sum()
        u = float(rng.uniform(0.0, 1.0))
        if abs(u - p1) < 1e-3:
            u = min(p1 + 2e-3, 0.999)
        b = u < p1
        w = np.where(one == b, w, 0.0)
        gates.append((("MEASURE", "RESET")[int(rng.integers(2))], (q,), u))
    return psi, gates


CASES = [(1, [0]), (2, [1]), (12, [0]), (13, [12]), (20, [3]),
         (10, [9, 8]), (12, [8, 11]), (12, [11, 9, 10]), (17, [8, 16]), (19, [18, 8]), (20, [13, 11]),
         (18, [10, 11, 12, 13, 14, 15, 16, 17]), (20, list(range(19, 7, -1))), (21, list(range(9, 21)))]


@pytest.mark.parametrize("n,qs", CASES)
def test_masses_and_decisions(ctx, n, qs):
    from paper_2609_23664_amd import binding as B
    import torch
    print("[gpu-case] masses", n, qs, flush=True)
    st = B.State(ctx, n, 3)
    want = []
    for k in range(3):
        psi, gates = _case(n, qs, 100 * n + k)
        st.buf[k].copy_(torch.from_numpy(psi))
        want.append((psi, gates))
    B.run_suffix_batch(ctx, None, [g for _, g in want], st, [0, 1, 2])
    got = B.outcomes(ctx).reshape(3, len(qs))
    for k, (psi, gates) in enumerate(want):
        ref = psi.astype(np.complex128)
        outs = [oracle._measure(ref, n, q[0], u, kind == "RESET") for kind, q, u in gates]
        assert list(got[k]) == outs, k
        s = st.host(k).astype(np.complex128)
        f = abs(np.vdot(ref, s)) ** 2 / (np.vdot(ref, ref).real * np.vdot(s, s).real)
        assert 1.0 - f <= 1e-6, k
        assert abs(np.vdot(s, s).real - 1.0) <= 1e-5, k
    st.free()

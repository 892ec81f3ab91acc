"""Expectation sums at the edges of their kernels: fewer and more terms than
waves, more than the 1,024 terms the final sum holds at a time, one and many
partial rows, states below 10 qubits. Against the oracle on the device's own
FP32 amplitudes: FP64 sums of at most 512 products below 10 qubits (2e-13 of
the coefficient sum), FP32 sums of 8 products a thread above (1.1e-6)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2609_23664_amd import binding as B
    return B.Ctx(0)


@pytest.mark.parametrize("n,count", [(1, 1), (3, 17), (9, 9), (9, 1025), (10, 1), (12, 1030), (16, 33), (18, 16)])
def test_expectation_term_edges(ctx, n, count):
    import torch
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] expectation edges", n, count, flush=True)
    rng = np.random.default_rng(31 * n + count)
    terms = []
    for _ in range(count):
        x, z = int(rng.integers(0, 1 << n)), int(rng.integers(0, 1 << n))
        if n > 9:   # X/Y support of at most 4 qubits
            keep = sum(1 << int(q) for q in rng.choice(n, size=4, replace=False))
            x &= keep
        terms.append((float(rng.standard_normal()), x, z))
    st = B.State(ctx, n, 2)
    v = (rng.standard_normal((2, 1 << n)) + 1j * rng.standard_normal((2, 1 << n))).astype(np.complex64)
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    st.buf.copy_(torch.from_numpy(v))
    e = st.expect(0, 2, terms)
    scale = sum(abs(c) for c, _, _ in terms)
    for k in range(2):
        ref = oracle.expect(v[k].astype(np.complex128), n, terms)
        assert abs(e[k] - ref) <= (2e-13 if n < 10 else 1.1e-6) * scale, k
    st.free()

"""Sampler at the edges of its kernels: states of less than one sub-chunk (64
amplitudes) and one chunk (1,024), one to more than 16,384 chunk sums (one
scan block and two), draws that do not fill a workgroup. Against the CDF of
the device's own FP32 amplitudes in extended precision: the index is the
smallest with CDF > u * total up to the FP64 rounding of the running sum (at
most about 150 additions and 2^5 scan blocks on a path: 1e-13 of the total)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2609_23664_amd import binding as B
    return B.Ctx(0)


def _splitmix(x):
    m = np.uint64
    with np.errstate(over="ignore"):
        x = x + m(0x9E3779B97F4A7C15)
        x = (x ^ (x >> m(30))) * m(0xBF58476D1CE4E5B9)
        x = (x ^ (x >> m(27))) * m(0x94D049BB133111EB)
    return x ^ (x >> m(31))


@pytest.mark.parametrize("n,slots,shots", [(1, 3, 5), (2, 2, 17), (5, 2, 33), (6, 1, 16), (8, 3, 50), (10, 2, 100),
                                           (11, 5, 7), (14, 2, 129), (20, 2, 1000), (21, 1, 1), (24, 1, 1024),
                                           (25, 1, 300)])
def test_sampler_level_edges(ctx, n, slots, shots):
    import torch
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] sampler edges", n, slots, shots, flush=True)
    rng = np.random.default_rng(n)
    st = B.State(ctx, n, slots)
    base, seed = 3, 77 + n
    states = []
    for k in range(slots):
        v = (rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)).astype(np.complex64)
        v[rng.random(1 << n) < 0.3] = 0.0
        v[0] += 0.5
        states.append(v)
        st.buf[k].copy_(torch.from_numpy(v))
    got = st.sample(0, slots, seed, base, shots)
    for k, v in enumerate(states):
        p = v.real.astype(np.float64) ** 2 + v.imag.astype(np.float64) ** 2
        cdf = np.cumsum(p.astype(np.longdouble))
        ctr = (np.uint64(base + k) << np.uint64(32)) + np.arange(shots, dtype=np.uint64)
        u = (_splitmix(np.uint64(seed) ^ ctr) >> np.uint64(11)).astype(np.float64) * 2.0 ** -53
        t = u * np.longdouble(cdf[-1])
        i = got[k].astype(np.int64)
        eps = np.longdouble(1e-13) * cdf[-1]
        assert np.all(p[i] > 0.0)
        assert np.all(cdf[i] > t - eps)
        assert np.all(np.where(i > 0, cdf[np.maximum(i - 1, 0)], 0.0) <= t + eps)
    st.free()

"""Interpreted pass kernels over every tile size (their workgroup size and LDS
bytes are launch arguments): one and several tiles, with and without a
renormalisation, several tasks. Bitwise equal to the generated kernels (the
same operations in the same order), and the oracle's state within the FP32
bar."""
import numpy as np
import pytest

import oracle
from tests.test_jit_host import _random_gates

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,tile", [(10, 10), (11, 10), (11, 11), (13, 12), (13, 13), (15, 13), (14, 14), (16, 14)])
def test_interpreted_tile_sizes(n, tile):
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] interpreted tiles", n, tile, flush=True)
    ctx = B.Ctx(0)
    ctx.set_option(B.QW_OPT_TILE_BITS, tile)
    lists = [_random_gates(n, 300 + n + k, 60) for k in range(3)]
    got = []
    for jit in (0, 2):
        ctx.set_option(B.QW_OPT_JIT, jit)
        st = B.State(ctx, n, 3)
        st.reset()
        B.run_suffix_batch(ctx, None, lists, st, [0, 1, 2])
        got.append([st.host(k).copy() for k in range(3)])
        st.free()
    for k in range(3):
        assert np.array_equal(got[0][k].view(np.uint32), got[1][k].view(np.uint32)), k
        ref = oracle.simulate(n, lists[k])
        assert 1.0 - oracle.fidelity(got[0][k].astype(np.complex128), ref) <= 1e-6, k

"""Expectation rows swept tile by tile (few states): the bits of the ways that
sweep whole rows, which are the interpreted reducers, a persistent launch for
the terms inside the last pass, and a context without room for the values per
tile. Tile counts from 2 (never split) to the largest split and past it, 1 to
50 terms, several states."""
import numpy as np
import pytest

from workloads import gen

pytestmark = pytest.mark.gpu


def _terms(n, count, seed):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(count):
        x, z = (int(v) for v in rng.integers(0, 1 << n, 2))
        keep = int(rng.integers(0, 1 << n)) & int(rng.integers(0, 1 << n))
        out.append((float(rng.normal()), x & keep, z & keep))
    return out


@pytest.mark.parametrize("n,tile,slots", [(11, 10, 3), (12, 10, 1), (12, 10, 5), (13, 11, 2), (17, 14, 6), (16, 14, 1),
                                          (14, 10, 16), (14, 10, 17), (20, 14, 1), (18, 10, 1), (19, 10, 1)])
@pytest.mark.parametrize("count", [1, 8, 9, 50])
def test_reducers_bits(n, tile, slots, count):
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] row sums", n, tile, slots, count, flush=True)
    ctx = B.Ctx(0)
    ctx.set_option(B.QW_OPT_TILE_BITS, tile)
    st = B.State(ctx, n, slots)
    st.reset()
    w = gen.small_vqe(n, 1, 1, slots, 1, seed=n)
    for s in range(slots):
        st.apply(s, w.task_gates(s))
    terms = _terms(n, count, 31 * n + count)
    got = []
    for jit in (0, 2):
        ctx.set_option(B.QW_OPT_JIT, jit)
        got.append(np.array(st.expect(0, slots, terms)))
    ctx.set_option(B.QW_OPT_DEVICE_MEM_CAP, slots * (8 << n) + (3 << 20))
    got.append(np.array(st.expect(0, slots, terms)))
    for g in got[1:]:
        assert np.array_equal(got[0].view(np.uint64), g.view(np.uint64))


@pytest.mark.parametrize("n,tile,tasks", [(15, 14, 3), (16, 14, 2), (17, 14, 6), (13, 10, 9), (16, 11, 8), (14, 10, 20)])
@pytest.mark.parametrize("count", [3, 20, 40])
def test_fused_bits(n, tile, tasks, count):
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] fused row sums", n, tile, tasks, count, flush=True)
    w = gen.small_vqe(n, 1, 2, tasks, count, seed=7 + n)
    got = []
    for persistent in (0, 1):
        ctx = B.Ctx(0)
        ctx.set_option(B.QW_OPT_JIT, 2)
        ctx.set_option(B.QW_OPT_TILE_BITS, tile)
        ctx.set_option(B.QW_OPT_PERSISTENT, persistent)
        st = B.State(ctx, n, tasks)
        st.reset()
        e = B.run_suffix_batch(ctx, None, [w.task_gates(t) for t in range(tasks)], st, list(range(tasks)),
                               terms=w.terms)
        got.append(np.array(e))
        st.free()
    assert np.array_equal(got[0].view(np.uint64), got[1].view(np.uint64))

"""Calls whose number of states crosses the last-level cache take other cache
policies, and so other generated kernels of the same structure: the one at hand
stands in, with the same bits, and nothing is compiled until its work has paid
for it. Counted by qw_jit_stats with an empty disk cache."""
import pytest
import torch

from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _cache(tmp_path, monkeypatch):
    monkeypatch.setenv("QW_JIT_CACHE", str(tmp_path / "jit"))


def _compiled(B):
    s = B.jit_stats()
    return s["compiled"] + s["disk_hits"]


def _ctx(B, jit, tile=14):
    ctx = B.Ctx(0)
    ctx.set_option(B.QW_OPT_JIT, jit)
    ctx.set_option(B.QW_OPT_LAYOUT, 0)   # one pass structure for one state and for many
    ctx.set_option(B.QW_OPT_TILE_BITS, tile)
    return ctx


def _layer(n, seed, turn):
    """One layer whose structure the seed picks (no other test's kernels)."""
    g = gen.rng(seed, 3)
    a = gen.random_angles(gen.rng(turn, 4), 3 * n)
    out = [("RY", (q,), a[q]) for q in range(n)] + [("RZ", (q,), a[n + q]) for q in range(n)]
    return out + [("CNOT", tuple(int(x) for x in g.choice(n, 2, replace=False)), 0.0) for _ in range(n)] + \
        [("RY", (q,), a[2 * n + q]) for q in range(n)]


@pytest.mark.parametrize("jit,first", [(2, "one"), (2, "many"), (1, "one")])
def test_crossing_compiles_nothing(jit, first):
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] stand-in kernels", jit, first, flush=True)
    # 264 MiB of states, or 528 (tiered: the batch alone passes the threshold of 4,096 tiles)
    n, k = 18, 132 if jit == 2 else 264
    gates = B.GateArray(_layer(n, 40 + 2 * jit + (first == "many"), 1))
    ctx = _ctx(B, jit)
    st = B.State(ctx, n, k + 1)

    def one():
        for _ in range(300 if jit == 1 else 1):   # (tiered: past the threshold)
            st.reset()
            st.apply(k, gates)

    def many():
        st.reset()
        B.run_suffix_batch(ctx, None, [gates] * k, st, list(range(k)))

    c0 = _compiled(B)
    (one if first == "one" else many)()
    c1 = _compiled(B)
    assert c1 > c0
    a = st.buf[k if first == "one" else 0].clone()
    (many if first == "one" else one)()
    ctx.sync()
    assert _compiled(B) == c1
    for s in range(k) if first == "one" else [k]:
        assert torch.equal(st.buf[s], a), s
    # a graph keeps its kernels, so a recording takes the right ones
    st.reset()
    ctx.begin_graph()
    (many if first == "one" else one)()
    g = ctx.end_graph()
    if jit == 2:
        assert _compiled(B) > c1
    for _ in range(2):
        g.replay()
        ctx.sync()
        assert torch.equal(st.buf[0 if first == "one" else k], a)
    g.free()
    st.free()


def test_stand_in_is_replaced_when_it_has_paid():
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] stand-in replaced", flush=True)
    n = 24
    # one pass with runs of 1,024 amplitudes: written through, for many states streamed
    gates = [(g, tuple(q if q < 10 else q + 10 for q in qs), x) for g, qs, x in _layer(14, 61, 1)]
    assert len(B.plan_describe(n, gates, 14)["passes"]) == 1
    gates = B.GateArray(gates)
    ctx = _ctx(B, 2)
    st = B.State(ctx, n, 3)
    st.apply(0, gates)
    c1, ref = _compiled(B), st.buf[0].clone()
    st.reset()

    def batch():
        B.run_suffix_batch(ctx, None, [gates] * 3, st, [0, 1, 2])   # 384 MiB

    batch()
    assert _compiled(B) == c1
    for s in range(3):
        assert torch.equal(st.buf[s], ref)
    calls = (1 << 40) // (3 << n)   # of the pass until its stand-in has paid
    for i in range(calls + 2):
        batch()
        if i % 2000 == 0:
            ctx.sync()
            assert i > calls - 2 or _compiled(B) == c1, i
    assert _compiled(B) == c1 + 1
    st.reset()
    batch()
    ctx.sync()
    for s in range(3):
        assert torch.equal(st.buf[s], ref)
    st.free()


def test_split_batch_keeps_one_policy():
    """A batch that the second-buffer cap splits into a large and a small part
    is one call: it compiles each structure once."""
    from paper_2609_23664_amd import binding as B
    from tests.test_gpu_relabel import _ladder_circuit
    import numpy as np
    print("[gpu-case] split batch", flush=True)
    n, k = 20, 34
    gates = B.GateArray(_ladder_circuit(n, np.random.default_rng(977), 3))
    passes = B.plan_describe(n, _ladder_circuit(n, np.random.default_rng(977), 3), 14)["passes"]
    assert any(p["out_cx"] for p in passes)
    ctx = _ctx(B, 2)
    ctx.set_option(B.QW_OPT_SECOND_BUFFER_CAP, 32 * (8 << n))   # 32 states (512 MiB with them), then 2
    st = B.State(ctx, n, k)
    c0 = _compiled(B)
    B.run_suffix_batch(ctx, None, [gates] * k, st, list(range(k)))
    ctx.sync()
    assert _compiled(B) - c0 <= len(passes)
    for s in range(1, k):
        assert torch.equal(st.buf[s], st.buf[0]), s
    st.free()

"""Recorded batches whose pass structures run as parallel branches of the graph
over three and more passes: branches that go on without a join, ones that meet
in a common later pass and part again, and ones that end after different counts
of passes. Replays give the bits of the direct calls. The plans' passes are
checked on the host and the graph's nodes counted, so that the lists keep the
shape that they are here for."""
import json

import numpy as np
import pytest
import torch

from paper_2609_23664_amd import binding as B

TILE = 10


def _block(qs, seed):
    """Rotations and CZs along qs and back: one pass over these qubits, more
    over any other set. The angles are the seed's."""
    g = np.random.default_rng(seed)
    out = []
    way = list(qs) + list(qs)[-2::-1]
    for a, b in zip(way, way[1:]):
        out += [("RY", (a,), float(g.uniform(0.1, 6.2))), ("RZ", (a,), float(g.uniform(0.1, 6.2))),
                ("CZ", (a, b), 0.0), ("RY", (b,), float(g.uniform(0.1, 6.2)))]
    return out


def _low(kind, seed):
    # from qubit 0 on: nothing of it fits a pass over the high qubits before
    return _block([0] + [int(q) for q in 1 + np.random.default_rng(90 + kind).permutation(TILE - 1)], seed)


def _high(n, kind, seed):
    # from the highest qubit on: nothing of it fits a pass over the low qubits before
    order = np.random.default_rng(70 + kind).permutation(TILE - 1)
    return _block([n - 1] + [n - 2 - int(q) for q in order], seed)


def _lists(n, shape):
    """Gate lists of a batch, two tasks of each structure."""
    parts = {
        # three structures that share no pass
        "apart": [[0, 0, 1], [1, 1, 2], [2, 2, 3, 3]],
        # common middle pass (low kinds differ before and after it)
        "meet": [[0, 0, 1], [1, 0, 2], [2, 0, 3]],
        # two share an early pass and part
        "part": [[0, 0, 1], [0, 0, 2], [0, 1, 3]],
        # they end after one, three and five passes
        "unequal": [[0], [1, 0, 1], [2, 1, 3, 0, 4]],
        # some meet, one goes on alone
        "mixed": [[0, 0, 1, 0, 2], [1, 0, 2, 1, 3], [2, 1, 3, 1, 4], [3, 1, 4]],
    }[shape]
    out = []
    for rep in range(2):
        for s, kinds in enumerate(parts):
            gates = []
            for i, k in enumerate(kinds):
                seed = 1000 * rep + 100 * s + i
                gates += _low(k, seed) if i % 2 == 0 else _high(n, k, seed)
            out.append(gates)
    return out


def _steps(n, lists):
    """Per pass index: the structure of each list's pass (None where it has ended)."""
    plans = []
    for gates in lists:
        passes = B.plan_describe(n, gates, TILE)["passes"]
        for p in passes:
            assert not p["norm_out"] and not p["out_cx"]
            for op in p["ops"]:
                op.pop("m")
        plans.append([json.dumps(p, sort_keys=True) for p in passes])
    most = max(len(p) for p in plans)
    return [[p[k] if k < len(p) else None for p in plans] for k in range(most)]


SHAPES = ["apart", "meet", "part", "unequal", "mixed"]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("n", [15, 17])
def test_lists_have_the_shape(n, shape):
    lists = _lists(n, shape)
    steps = _steps(n, lists)
    assert len(steps) >= 3
    half = len(lists) // 2
    kinds = [len(set(s) - {None}) for s in steps]
    assert all(s[:half] == s[half:] for s in steps)     # two tasks of each structure
    print(shape, n, kinds, [sum(x is None for x in s) for s in steps])
    if shape in ("apart", "unequal"):
        # a structure's pass is nobody else's: the branches go on unjoined
        assert all(k == len(set(s[:half]) - {None}) and len([x for x in s[:half] if x]) == k
                   for s, k in zip(steps, kinds)) and kinds[0] > 1 and kinds[1] > 1
    if shape == "unequal":
        assert len({sum(s[t] is not None for s in steps) for t in range(half)}) == half
    if shape == "meet":
        assert kinds[0] == 3 and 1 in kinds[1:-1] and kinds[-1] == 3
    if shape == "part":
        assert 2 in kinds[:2] and kinds[-1] == 3
    if shape == "mixed":
        assert any(1 < k < sum(x is not None for x in s[:half]) for s, k in zip(steps, kinds))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("n", [15, 17])
def test_replays_give_the_direct_bits(n, shape):
    print("[gpu-case] graph branch paths", n, shape, flush=True)
    lists = _lists(n, shape)
    steps = _steps(n, lists)
    k = len(lists)
    ctx = B.Ctx(0)
    # (the plans that _steps describes: from a source state, with layouts)
    for opt, value in ((B.QW_OPT_JIT, 2), (B.QW_OPT_TILE_BITS, TILE), (B.QW_OPT_LAYOUT, 2)):
        ctx.set_option(opt, value)
    first, st, other = B.State(ctx, n, 1), B.State(ctx, n, k), B.State(ctx, n, k)
    first.buf.copy_(torch.view_as_complex(torch.randn(1, 1 << n, 2, device="cuda")))
    torch.cuda.synchronize()
    src = first.snapshot(0, b"s" * 32, B.QW_SNAP_FREEZE)

    def work(dst):
        B.run_suffix_batch(ctx, [src] * k, lists, dst, list(range(k)))

    work(st)
    ctx.sync()
    ref = st.buf.clone()
    ctx.begin_graph()
    work(st)
    g = ctx.end_graph()
    assert g.nodes() == sum(len(set(s) - {None}) for s in steps)
    for rep in range(6):
        st.buf.zero_()
        other.buf.zero_()
        torch.cuda.synchronize()
        g.replay()
        if rep % 2:
            work(other)   # the context's own calls between the replays
        ctx.sync()
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(st.buf), torch.view_as_real(ref)), rep
    g.free()
    src.free()
    for s in (other, st, first):
        s.free()

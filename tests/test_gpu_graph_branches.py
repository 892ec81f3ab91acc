"""Recorded batches of several pass structures (parallel branches of the
graph): replays give the bits of the direct calls. The structures stay apart
over their passes, meet in a common later pass, or end after different counts
of passes; and renormalised ones join at each pass."""
import numpy as np
import pytest
import torch

from tests.test_jit_host import _random_gates

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kinds,jit", [(1, 2), (2, 2), (3, 2), (5, 2), (3, 0), (2, 1)])
@pytest.mark.parametrize("n", [15, 17])
def test_branches_replay_bits(n, kinds, jit):
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] graph branches", n, kinds, jit, flush=True)
    ctx = B.Ctx(0)
    ctx.set_option(B.QW_OPT_JIT, jit)
    k = 4 * kinds + 1
    lists = [_random_gates(n, 400 + t % kinds, 12 * (1 + t % kinds)) for t in range(k)]
    follow = [_random_gates(n, 500 + t % 2, 40) for t in range(k)]
    st = B.State(ctx, n, k)

    def work():
        st.reset()
        B.run_suffix_batch(ctx, None, lists, st, list(range(k)))
        B.run_suffix_batch(ctx, None, follow, st, list(range(k)))

    work()
    torch.cuda.synchronize()
    ref = st.buf.clone()
    ctx.begin_graph()
    work()
    g = ctx.end_graph()
    for rep in range(4):
        st.buf.zero_()
        torch.cuda.synchronize()
        g.replay()
        ctx.sync()
        torch.cuda.synchronize()
        assert torch.equal(st.buf.view(torch.float32), ref.view(torch.float32)), rep
    g.free()
    st.free()

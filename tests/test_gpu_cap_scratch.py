"""Under a device-memory cap an expectation over few states keeps its scratch
small: a state that fits beside the first one's expectations is not refused,
and the values are those of a context without a cap (rows swept tile by tile
there)."""
import pytest
import torch

from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("recorded", [0, 1])
def test_second_state_fits(fused, recorded):
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] expectation scratch under a cap", fused, recorded, flush=True)
    n, values = 17, []
    w = gen.small_vqe(n, 1, 2, 1, 50, seed=5)
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    for cap in (0, 3 << 20):   # a state is 1 MiB, values per tile would be 1.6 MB
        ctx = B.Ctx(0)
        ctx.set_option(B.QW_OPT_JIT, 2)
        ctx.set_option(B.QW_OPT_FUSED_EPILOGUE, fused)
        ctx.set_option(B.QW_OPT_DEVICE_MEM_CAP, cap)
        st = B.State(ctx, n, 1)
        st.apply(0, w.prefix)
        if recorded:
            ctx.begin_graph()
        B.run_suffix_batch(ctx, None, [w.suffixes[0]], st, [0], terms=w.terms, out_dev=out)
        g = ctx.end_graph() if recorded else None
        if g:
            g.replay()
        ctx.sync()
        second = B.State(ctx, n, 1)
        values.append((out.cpu().tolist(), st.buf.cpu()))
        if g:
            g.free()
        second.free()
        st.free()
    assert values[0][0] == values[1][0]
    assert torch.equal(torch.view_as_real(values[0][1]), torch.view_as_real(values[1][1]))

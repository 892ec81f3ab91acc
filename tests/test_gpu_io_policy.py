"""Cache policies of the generated passes: a batch larger than the last-level
cache (other policies by the tiles' run lengths) gives the bits of the
interpreted kernels, which have none, and of one-state calls, in place, with
permuted layouts and from a shared snapshot."""
import pytest
import torch

from tests.test_jit_host import _random_gates

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [10, 12, 14])
@pytest.mark.parametrize("layout,snap,stream", [(0, 0, 1), (2, 0, 1), (2, 0, 0), (1, 1, 1)])
def test_large_batch_bits(tile, layout, snap, stream):
    from paper_2609_23664_amd import binding as B
    n, k = 18, 132  # 264 MiB of states
    print("[gpu-case] cache policies", tile, layout, snap, stream, flush=True)
    ctx = B.Ctx(0)
    ctx.set_option(B.QW_OPT_TILE_BITS, tile)
    ctx.set_option(B.QW_OPT_LAYOUT, layout)
    ctx.set_option(B.QW_OPT_STREAM_LOADS, stream)
    gates = B.GateArray(_random_gates(n, 7 + tile, 50))
    pre = B.GateArray(_random_gates(n, 8, 30))
    st = B.State(ctx, n, k + 1)
    got = []
    for mode in ("generated", "interpreted", "one by one"):
        ctx.set_option(B.QW_OPT_JIT, 0 if mode == "interpreted" else 2)
        st.reset()
        st.apply(0, pre)
        src = st.snapshot(0, b"p" * 32, B.QW_SNAP_FREEZE) if snap else None
        batch = [range(1, k + 1)] if mode != "one by one" else [[1], [k]]
        for b in batch:
            B.run_suffix_batch(ctx, [src] * len(b) if snap else None, [gates] * len(b), st, list(b))
        torch.cuda.synchronize()
        if src:
            src.free()
        got.append(st.buf[1].clone())
        if mode != "one by one":
            assert all(torch.equal(st.buf[s], st.buf[1]) for s in range(2, k + 1)), mode
        else:
            assert torch.equal(st.buf[k], st.buf[1])
    assert torch.equal(got[0], got[1])
    assert torch.equal(got[0], got[2])

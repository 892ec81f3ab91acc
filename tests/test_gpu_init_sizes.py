"""Reset of states at the sizes where its kernel changes (256 MiB, 1 and 4 GiB)
and beside them. Exact."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,slots", [(25, 1), (18, 129), (24, 3), (26, 2), (20, 127), (27, 1), (20, 129), (25, 5),
                                     (28, 1), (20, 511), (29, 1), (20, 513)])
def test_reset_sizes(n, slots):
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] reset sizes", n, slots, (slots * 8 << n) >> 20, "MiB", flush=True)
    ctx = B.Ctx(0)
    st = B.State(ctx, n, slots)
    st.buf.fill_(complex(2.0, -3.0))
    st.reset()
    torch.cuda.synchronize()
    assert bool((st.buf[:, 0] == 1.0).all())
    st.buf[:, 0] = 0.0
    assert torch.count_nonzero(torch.view_as_real(st.buf)).item() == 0
    st.free()

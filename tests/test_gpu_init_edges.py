"""Reset of consecutive slots to |0>: the smallest states, sizes around a
workgroup's share, both store policies (up to 256 MiB and above), and the
slots beside the range untouched. Exact."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,slots,first,count", [(1, 5, 1, 3), (2, 3, 0, 3), (9, 7, 2, 5), (10, 3, 1, 1), (11, 4, 1, 2),
                                                 (12, 3, 0, 2), (17, 3, 1, 2), (25, 2, 0, 1), (25, 3, 1, 2), (26, 1, 0, 1)])
def test_reset_range(n, slots, first, count):
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] reset", n, slots, first, count, flush=True)
    ctx = B.Ctx(0)
    st = B.State(ctx, n, slots)
    st.buf.fill_(complex(2.0, -3.0))
    st.reset(first, count)
    torch.cuda.synchronize()
    for s in range(slots):
        if first <= s < first + count:
            assert st.buf[s, 0].item() == 1.0 and torch.count_nonzero(torch.view_as_real(st.buf[s])).item() == 1
        else:
            assert bool((st.buf[s] == complex(2.0, -3.0)).all())
    st.free()

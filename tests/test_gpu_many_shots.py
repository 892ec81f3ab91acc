"""Draws of many shots (one thread each) against draws of few (8 lanes each):
shot k of a slot depends on the seed, the slot and k alone, so a call of few
shots returns the beginning of a call of many, over states whose mass is spread,
close together, at either end, in few amplitudes, and none; and many draws of a
concentrated state do not cost what a spread one costs."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LINE = 49152   # draws of a call, the last one with 8 lanes a shot


def _fill(st, n, slots, kind):
    g = torch.Generator(device="cuda").manual_seed(n)
    st.buf.zero_()
    if kind == "spread":
        st.buf.copy_(torch.view_as_complex(torch.randn(slots, 1 << n, 2, device="cuda", generator=g)))
    elif kind == "first":
        st.buf[:, 0] = 1.0
    elif kind == "last":
        st.buf[:, -1] = 1.0
    elif kind == "few":
        st.buf[:, torch.randint(0, 1 << n, (9,), device="cuda", generator=g)] = 1.0 / 3
    elif kind == "decay":
        i = torch.arange(1 << n, device="cuda")
        st.buf.copy_((2.0 ** (-0.25 * (i % 4001))).to(torch.complex64).expand(slots, -1))
    torch.cuda.synchronize()


@pytest.mark.parametrize("kind", ["spread", "first", "last", "few", "decay", "zero"])
@pytest.mark.parametrize("n,slots", [(1, 3), (3, 2), (5, 1), (6, 1), (7, 5), (9, 2), (10, 3), (13, 7), (17, 2), (21, 1)])
def test_few_are_the_beginning_of_many(n, slots, kind):
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] many shots", n, slots, kind, flush=True)
    ctx = B.Ctx(0)
    st = B.State(ctx, n, slots)
    _fill(st, n, slots, kind)
    few = LINE // slots
    for many in (few + 1, 3 * few + 77):
        a = torch.empty(slots * few, dtype=torch.int32, device="cuda")
        b = torch.empty(slots * many, dtype=torch.int32, device="cuda")
        st.sample(0, slots, 11, 5, few, out_dev=a)
        st.sample(0, slots, 11, 5, many, out_dev=b)
        ctx.sync()
        a, b = a.view(slots, few), b.view(slots, many)
        assert torch.equal(a, b[:, :few])
        assert int(b.min()) >= 0 and int(b.max()) < 1 << n
        if kind != "zero":
            amp = torch.gather(st.buf, 1, b.long())
            assert bool((amp.abs() > 0).all())
        else:
            assert bool((b == b[0, 0]).all())
    st.free()


@pytest.mark.parametrize("kind", ["first", "last"])
def test_concentrated_states_are_cheap(kind):
    """2^22 draws of 64 14-qubit states: 454 (first) and 468 us (last) when all
    64 amplitudes were added for every shot, 39 and 108 like this."""
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] many shots, time", kind, flush=True)
    n, slots, shots = 14, 64, 65536
    ctx = B.Ctx(0)
    st = B.State(ctx, n, slots)
    _fill(st, n, slots, kind)
    out = torch.empty(slots * shots, dtype=torch.int32, device="cuda")
    times = []
    for _ in range(8):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        st.sample(0, slots, 1, 0, shots, out_dev=out)
        e[1].record()
        e[1].synchronize()
        times.append(e[0].elapsed_time(e[1]) * 1e3)
    print("  us", round(min(times), 1), flush=True)
    assert min(times) < 250
    st.free()

"""Plan uploads and host outputs: calls enqueued without a wait between them
reuse the staging slots (blobs below and above 16 KiB and 1 MiB), and every
state must be bitwise the one of the same call followed by a wait; host
outputs below and above the size written straight to pinned memory must equal
the device outputs bitwise."""
import numpy as np
import pytest

from workloads import gen

pytestmark = pytest.mark.gpu


def _gates(n, layers, seed):
    g = gen.rng(seed, 1)
    out = []
    for _ in range(layers):
        out += gen.hea_layer(n, gen.random_angles(g, 2 * n))
    return out


@pytest.mark.parametrize("n,layers,calls", [(11, 1, 120), (12, 20, 40), (12, 6, 70)])
def test_back_to_back_uploads(n, layers, calls):
    import torch
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] staging", n, layers, calls, flush=True)
    lists = [_gates(n, 1 + k % layers, 500 + k) for k in range(calls)]
    states = []
    for wait in (True, False):
        ctx = B.Ctx(0)
        st = B.State(ctx, n, calls)
        torch.cuda.synchronize()
        for k, g in enumerate(lists):
            st.apply(k, g)
            if wait:
                ctx.sync()
        ctx.sync()
        states.append(st.buf.cpu().numpy().copy())
        st.free()
    assert np.array_equal(states[0].view(np.uint32), states[1].view(np.uint32))


def test_batch_blobs_above_one_mebibyte():
    import torch
    from paper_2609_23664_amd import binding as B
    n, T = 12, 256
    print("[gpu-case] staging of large batches", flush=True)
    ctx = B.Ctx(0)
    batches = [[_gates(n, 3, 1000 * b + t) for t in range(T)] for b in range(3)]
    ref, got = [], []
    for wait in (True, False):
        states = [B.State(ctx, n, T) for _ in batches]
        torch.cuda.synchronize()
        for st, b in zip(states, batches):
            B.run_suffix_batch(ctx, None, b, st, list(range(T)))
            st.apply(0, b[1])
            if wait:
                ctx.sync()
        ctx.sync()
        (ref if wait else got).extend(st.buf.cpu().numpy().copy() for st in states)
        for st in states:
            st.free()
    for a, b in zip(ref, got):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("shots", [100, 1 << 19, (1 << 19) + 1])
def test_host_output_equals_device_output(shots):
    import torch
    from paper_2609_23664_amd import binding as B
    print("[gpu-case] host output", shots, flush=True)
    ctx = B.Ctx(0)
    st = B.State(ctx, 11, 2)
    v = torch.view_as_complex(torch.randn(2, 1 << 11, 2, device="cuda"))
    st.buf.copy_(v)
    dev = torch.empty(2 * shots, dtype=torch.int32, device="cuda")
    st.sample(0, 2, 9, 0, shots, out_dev=dev)
    host = st.sample(0, 2, 9, 0, shots)
    assert np.array_equal(dev.cpu().numpy().view(np.uint32).reshape(2, shots), host)
    e = torch.empty(2, dtype=torch.float64, device="cuda")
    terms = [(0.5, 3, 5), (-1.25, 0, 9)]
    st.expect(0, 2, terms, out_dev=e)
    assert st.expect(0, 2, terms) == e.cpu().tolist()
    st.free()

"""Cost-model kernels at the edges of their row groups (16 rows a workgroup,
16 groups a sweep of the weight kernel): forward and gradient against the
BF16-mirrored oracle, with the bars of the larger batches (FP32 sums of at
most 2,000 products: 2e-5 and 1e-4)."""
import numpy as np
import pytest

from oracle import mlp_ref as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2609_23664_amd import binding
    return binding.Ctx(0)


@pytest.mark.parametrize("B", [1, 2, 15, 16, 17, 33, 256, 257, 2000])
def test_row_group_edges(ctx, B):
    import torch
    from paper_2609_23664_amd import costmodel as CM
    print("[gpu-case] mlp edges", B, flush=True)
    rng = np.random.default_rng(900 + B)
    n = B + 5
    x = rng.uniform(0, 1, size=(n, M.IN)).astype(np.float32)
    t = rng.normal(size=(n, M.OUT)).astype(np.float32)
    rows = rng.integers(0, n, size=B)
    p = CM.init_params(11)
    mlp = CM.MLP(ctx, params=p)
    p64, xb, tb = p.astype(np.float64), x[rows].astype(np.float64), t[rows].astype(np.float64)
    y = mlp.predict(x[rows])
    _, _, ref = M.forward(p64, xb, bf16_inputs=True)
    assert np.max(np.abs(y - ref)) <= 2e-5 * max(1e-6, np.max(np.abs(ref)))
    g = mlp.backward_rows(torch.tensor(x, device="cuda"), torch.tensor(t, device="cuda"), rows)
    g = g.cpu().numpy().astype(np.float64)
    gbf = M.backward(p64, xb, tb, bf16_inputs=True)
    assert np.linalg.norm(g - gbf) <= 1e-4 * np.linalg.norm(gbf)

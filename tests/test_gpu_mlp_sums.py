"""Sums over rows of the network's gradient."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [8192, 65536])
def test_gradient_sum_over_rows(m):
    """The gradient of m rows is the mean of those of its 1,024-row parts: a power of
    two of them, so every row's own terms round alike (the output gradient's scale
    differs by a power of two) and only the sums over rows differ.  Rounding the sum
    once to fp32 is at most 2^-24 of a component; partial sums of 256 rows added in
    fp32 came within 4.6e-8 of a matrix's norm."""
    import torch
    from oracle import mlp as OM
    from paper_2406_07441_amd import lskum as lk
    part = 1024
    rng = np.random.default_rng(0)
    X = torch.from_numpy(rng.uniform(-1, 1, (m, 5)).astype(np.float32)).cuda()
    T = (0.3 * torch.sin(np.pi * X[:, :4])).contiguous()
    net = lk.MLP(seed=3, max_rows=m)
    net.set_params((2 * net.get_params()).astype(np.float32))
    _, g = net.gradient(X, T)
    mean = sum(np.asarray(net.gradient(X[k:k + part], T[k:k + part])[1], np.float64)
               for k in range(0, m, part)) * (part / m)
    net.close()
    o = 0
    for name, shape in OM.SHAPES:
        k = int(np.prod(shape))
        e = np.linalg.norm(g[o:o + k] - mean[o:o + k]) / np.linalg.norm(mean[o:o + k])
        print(f"{m} rows, {name}: {e:.1e}")
        assert e <= (4.6e-8 if len(shape) > 1 and m == 8192 else 2.0 ** -24), name
        o += k

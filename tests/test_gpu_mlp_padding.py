"""Rows that only pad a training pass (a batch that is no multiple of 32)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lk():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07441_amd import lskum
    lskum.lib()
    return lskum


def _rows(n, bad):
    rng = np.random.default_rng(3)
    X = rng.uniform(-1, 1, (n, 5)).astype(np.float32)
    T = (0.3 * np.sin(np.pi * X[:, :4])).astype(np.float32)
    X[0] = bad
    return X, T


@pytest.mark.parametrize("bad", [np.nan, np.inf, 3e38])
@pytest.mark.parametrize("batch", [1, 31, 40])
def test_rows_that_are_not_drawn_do_not_matter(lk, bad, batch):
    """Row 0 of the data set is not finite (or overflows in layer 1) and is never
    drawn: the weights after training are those of the same data with a plain
    row 0."""
    import torch
    n, steps, seed = 100000, 3, 11
    out = []
    for first in (bad, 0.25):
        X, T = _rows(n, first)
        net = lk.MLP(seed=2, max_rows=64)
        hist, _ = net.train(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), steps, batch,
                            1e-3, seed=seed)
        out.append((hist, net.get_params()))
        net.close()
    assert np.isfinite(out[0][0]).all() and np.isfinite(out[0][1]).all()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


def test_a_row_of_the_batch_still_counts(lk):
    """A gradient over rows that hold a NaN is a NaN, padding or not."""
    import torch
    for m in (1, 33):
        X, T = _rows(m, np.nan)
        net = lk.MLP(seed=2, max_rows=64)
        loss, g = net.gradient(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda())
        assert np.isnan(loss) and np.isnan(g).any()
        net.close()

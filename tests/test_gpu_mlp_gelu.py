"""The forward pass's GELU: max(z, 0) - |z| Phi(-|z|) by a fit wherever a wavefront
holds a |z| beyond 1.4 and none beyond 4, with erff elsewhere and where the fit cannot
settle the bfloat16 rounding."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
UNITS = 4


@pytest.fixture(scope="module")
def lk():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07441_amd import lskum
    lskum.lib()
    return lskum


def _rows(z):
    """Features whose bfloat16 parts add up to z exactly (24 bits as 8 + 8 + 8)."""
    import torch
    X = torch.zeros((z.numel(), 5), dtype=torch.float32, device="cuda")
    rest = z.clone()
    for f in range(3):
        X[:, f] = rest.to(torch.bfloat16).float()
        rest -= X[:, f]
    assert not rest.any()
    return X


def _net(lk, rows, w2, w3, b1=()):
    """Units 0..3 in three lines: z = x0 + x1 + x2 + b1, then w2 and w3 (one weight
    each), outputs 0..3; every other weight is zero."""
    from oracle import mlp as OM
    th = {n: np.zeros(s, np.float32) for n, s in OM.SHAPES}
    th["b1"][:len(b1)] = b1
    for u in range(UNITS):
        th["W1"][u, :3] = 1.0
        th["W2"][u, u], th["W3"][u, u], th["W4"][u, u] = w2[u], w3[u], 1.0
    net = lk.MLP(max_rows=rows)
    net.set_params(np.concatenate([th[n].ravel() for n, _ in OM.SHAPES]))
    return net


@pytest.mark.parametrize("lo,hi,stride", [(1.4, 4.0, 1), (0.0, 1e30, 64)])
def test_fit_has_the_bits_of_erff(lk, lo, hi, stride):
    """Every float of 1.4 to 4 (waves that take the fit), and every 64th up to 1e30,
    both signs, as layer 1's z: the training pass takes erff everywhere, so its loss
    against the forward pass's outputs is exactly zero if all activations have the same
    bits (one weight a line: no sums to round; gelu is one to one on what layers 2 and
    3 get from the lines of weight -1, up to a rounding on the others)."""
    import torch
    ends = np.array([lo, hi], np.float32).view(np.int32)
    bits = torch.arange(int(ends[0]), int(ends[1]) + 1, stride, dtype=torch.int32, device="cuda")
    a = bits.view(torch.float32)
    a = torch.where(a < 1e-30, torch.zeros_like(a), a)  # parts would be subnormal
    z = torch.cat([a, -a])
    rows = 1 << 24
    net = _net(lk, rows, (1, -1, 4, -8), (1, 1, -2, 1))
    for k in range(0, z.numel(), rows):
        X = _rows(z[k:k + rows])
        Y = net.forward(X)
        loss, _ = net.gradient(X, Y)
        assert torch.isfinite(Y).all() and loss == 0.0, (k, loss)
    net.close()


def test_near_values_alone_and_in_mixed_waves(lk):
    """|z| up to 1.4 takes erff in a wavefront of its own and the fit beside larger
    values: the same bits (ties of the rounding are one value in 10,000)."""
    import torch
    m = 1 << 20
    z = torch.linspace(-1.4, 1.4, m, device="cuda")
    far = torch.full((m,), 3.0, device="cuda")
    both = torch.stack([z, far], 1).reshape(-1)
    net = _net(lk, 2 * m, (1, -1, 0.5, -0.5), (1, 1, 1, 1))
    alone = net.forward(_rows(z))
    mixed = net.forward(_rows(both))[::2]
    net.close()
    assert torch.equal(alone, mixed)


def test_activations_against_exact_gelu(lk):
    """Outputs of the lines against gelu in double precision: with |z| up to 8 in
    layer 1, each activation is a bfloat16 neighbour of what lies within 3e-7 |z| of
    gelu(z) (fp32 erff and products, 2^-24 |z| each, and the fit's interval)."""
    import torch
    from scipy.special import ndtr
    m = 1 << 18
    rng = np.random.default_rng(4)
    z = rng.uniform(-8, 8, m).astype(np.float32)
    z[np.abs(z) < 1e-3] = 0.5

    def bf16(a):
        return torch.from_numpy(np.asarray(a, np.float32)).to(torch.bfloat16).double().numpy()

    net = _net(lk, m, (1, -1, 4, -8), (1, 1, -2, 1))
    Y = net.forward(_rows(torch.from_numpy(z).cuda())).double().cpu().numpy()
    net.close()
    for u, (w2, w3) in enumerate(zip((1, -1, 4, -8), (1, 1, -2, 1))):
        lo = hi = z.astype(np.float64)
        for w in (w2, w3, 1):
            ends = []
            for s, v in ((-1, lo), (1, hi)):
                g = v * ndtr(v)
                ends += [bf16(g - 3e-7 * np.abs(v)), bf16(g + 3e-7 * np.abs(v))]
            lo, hi = np.minimum.reduce(ends) * w, np.maximum.reduce(ends) * w
            lo, hi = np.minimum(lo, hi), np.maximum(lo, hi)
        assert np.all((Y[:, u] >= lo) & (Y[:, u] <= hi)), u
        if u < 2:  # pinned to one value; line 2 and 3 end where gelu fades out
            assert np.mean(lo[np.abs(z) < 3] == hi[np.abs(z) < 3]) > 0.95, u

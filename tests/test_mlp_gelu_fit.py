"""The fit behind the network's activations (phi_lower in csrc/lskum_mlp.hip)."""
import os
import re

import numpy as np
import pytest
from scipy.special import erf, ndtr

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2406_07441_amd", "csrc", "lskum_mlp.hip")
F = np.float32


@pytest.fixture(scope="module")
def source():
    return open(SRC).read()


@pytest.fixture(scope="module")
def coef(source):
    body = source[source.index("float phi_lower"):source.index("exp2f(p)")]
    return [F(v) for v in re.findall(r"([-+]?\d+\.\d*(?:e[-+]\d+)?)f", body)]


def test_fit(coef):
    """Error relative to |z| as the generator states it, exactly 1/2 at 0, and falling
    beyond the fitted range."""
    assert len(coef) == 11 and coef[-1] == -1.0
    c = np.array(coef, np.float64)
    a = np.linspace(0, 6, 100001)
    assert np.abs(2.0 ** np.polyval(c, a) - ndtr(-a)).max() <= 2.5e-9
    assert np.all(np.diff(np.polyval(c, np.geomspace(6, 1e4, 10000))) < 0)


def test_interval(source, coef):
    """The two forms of gelu in fp32 steps (fused multiply-adds rounded once, erf and
    2^P rounded correctly) over every 29th float of [1e-4, 12]: apart by less than the
    interval that the kernel lays around its estimate, with a tenth to spare for
    device functions that round otherwise."""
    diff = float(re.search(r"kDiff = ([\d.e-]+)f", source).group(1))
    lo, hi = np.array([1e-4, 12.0], F).view(np.int32)
    worst = 0.0
    for bits in np.array_split(np.arange(lo, hi, 29, dtype=np.int32), 8):
        a = bits.view(F)
        p = np.full(a.shape, coef[0], F)
        for c in coef[1:]:
            p = (p.astype(np.float64) * a + np.float64(c)).astype(F)
        phi = np.exp2(p.astype(np.float64)).astype(F)
        for z in (a, -a):
            est = (np.maximum(z, 0) - a.astype(np.float64) * phi).astype(F)
            e = erf((z * F(0.70710678118654752)).astype(np.float64)).astype(F)
            g = (F(0.5) * z) * (F(1) + e)
            worst = max(worst, (np.abs(est.astype(np.float64) - g) / a).max())
    print(f"apart by {worst:.3e} |z|")
    assert worst <= 0.9 * diff

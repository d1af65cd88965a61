"""Dispatch rules of the solver kernels: where a launch takes another form by
size, both forms must give the same result."""
import numpy as np
import pytest

import oracle as O
from paper_2406_07441_amd import cloudgen as cg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lk():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07441_amd import lskum
    lskum.lib()
    return lskum


@pytest.mark.parametrize("precision,farfield", [(0, 0), (1, 0), (0, 1)])
def test_residual_forms_agree_bitwise(lk, precision, farfield):
    """Six conditions on clouds of 2,304 and 3,840 points (18,432 points: tiled
    residual) against single states (gathered residual): the same bits."""
    a = lk.Cloud(cg.ogrid(96, 24, r=1.12, t=0.12))
    b = lk.Cloud(cg.ogrid(128, 30, r=1.1, t=0.10, jitter_p=0.05, seed=3))
    conds = [(0, 0.5, 2.0), (1, 0.63, -1.0), (0, 0.7, 3.0), (1, 0.8, 1.0), (1, 0.4, 0.0), (0, 0.6, 1.0)]
    kw = dict(cfl=50.0, limiter=1, precision=precision, farfield=farfield)
    bat = lk.Batch([a, b], [c[0] for c in conds], [c[1] for c in conds], [c[2] for c in conds],
                   lk.default_params(**kw))
    for _ in range(3):
        bat.step_timed()
    for k, (ci, m, al) in enumerate(conds):
        st = lk.State([a, b][ci], m, al, lk.default_params(**kw))
        for _ in range(3):
            st.step(want_res=False)
        assert np.array_equal(bat.get_U(k), st.get_U()), k
        st.close()
    bat.close()


@pytest.mark.parametrize("nw,nk,lanes,gamma", [(258, 70, 1, 1.4), (258, 70, 2, 1.4), (258, 70, 4, 1.4),
                                               (258, 70, 8, 1.4), (258, 70, 2, 1.3), (96, 24, 2, 1.3)])
def test_residual_lanes_and_gamma(lk, nw, nk, lanes, gamma):
    """Tiled residual (18,060 points, the last tile of a band ragged) at every
    lane count, and gamma other than 1.4 in both forms, against the oracle at a
    transonic state with points beyond |S| = 1: the suite's bar of 1e-11."""
    cloud = cg.ogrid(nw, nk, jitter_p=0.04, seed=9)
    kw = dict(cfl=50.0, inner_iters=1, limiter=1, limiter_k=5.0)
    o = O.Oracle(cloud, mach=1.4, aoa_deg=1.0, gamma=gamma, **kw)
    st = lk.State(lk.Cloud(cloud), 1.4, 1.0,
                  lk.default_params(residual_lanes=lanes, gamma=gamma, **kw))
    U = o.free_stream()
    for _ in range(2):
        U = o.iteration(U)[0]
    st.set_U(U)
    R, res = st.residual()
    Ro, reso = o.residual(U)
    e = max(np.abs(R[v] - Ro[v]).max() / np.abs(Ro[v]).max() for v in range(4))
    print(f"residual {nw}x{nk} lanes {lanes} gamma {gamma}: {e:.2e}")
    assert e < 1e-11 and abs(res - reso) <= 1e-11 * reso

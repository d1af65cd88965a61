"""Forms of the solver kernels that no default launch of these sizes takes,
against those that it does: the same bits."""
import numpy as np
import pytest

from paper_2406_07441_amd import cloudgen as cg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lk():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07441_amd import lskum
    lskum.lib()
    return lskum


@pytest.mark.parametrize("qgrad_lanes", [0, 4])
@pytest.mark.parametrize("precision,farfield", [(0, 0), (1, 0), (0, 1)])
def test_tiled_batch_against_gathered_states(lk, precision, farfield, qgrad_lanes):
    """A batch of 18,432 points (288 tiles, two threads to a lane) against single
    states of 2,304 and 3,840 points that ask for two lanes (fewer than 256 tiles:
    gathered), with the q-derivative passes tiled and gathered."""
    a = lk.Cloud(cg.ogrid(96, 24, r=1.12, t=0.12))
    b = lk.Cloud(cg.ogrid(128, 30, r=1.1, t=0.10, jitter_p=0.05, seed=3))
    conds = [(0, 0.5, 2.0), (1, 0.63, -1.0), (0, 0.7, 3.0), (1, 0.8, 1.0), (1, 0.4, 0.0), (0, 0.6, 1.0)]
    kw = dict(cfl=50.0, limiter=1, precision=precision, farfield=farfield, qgrad_lanes=qgrad_lanes)
    bat = lk.Batch([a, b], [c[0] for c in conds], [c[1] for c in conds], [c[2] for c in conds],
                   lk.default_params(**kw))
    for _ in range(3):
        bat.step_timed()
    for k, (ci, m, al) in enumerate(conds):
        st = lk.State([a, b][ci], m, al, lk.default_params(residual_lanes=2, **kw))
        for _ in range(3):
            st.step(want_res=False)
        assert np.array_equal(bat.get_U(k), st.get_U()), k
        st.close()
    bat.close()

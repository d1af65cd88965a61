"""Host copies of fields from several threads at once."""
from concurrent.futures import ThreadPoolExecutor

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


@pytest.mark.parametrize("nw,nk", [(20, 6), (320, 103), (512, 256)])
def test_conditions_read_by_a_thread_pool(lk, nw, nk):
    """Six conditions of a batch, and one state's field and increment, copied by
    four threads: every call gets its own field (one chunk, two, four and more)."""
    c = lk.Cloud(cg.ogrid(nw, nk))
    b = lk.Batch([c], [0] * 6, [0.3 + 0.05 * k for k in range(6)], [1.0] * 6, lk.default_params(cfl=20.0))
    b.step_timed()
    st = lk.State(c, 0.5, 1.0, lk.default_params(cfl=20.0))
    st.step()
    jobs = [lambda k=k: b.get_U(k) for k in range(6)] + [st.get_U, st.get_dU]
    alone = [j() for j in jobs]
    assert all(not np.array_equal(alone[0], a) for a in alone[1:])
    with ThreadPoolExecutor(4) as pool:
        for _ in range(5):
            for a, g in zip(alone, pool.map(lambda j: j(), jobs)):
                assert np.array_equal(a, g)
    st.close()
    b.close()

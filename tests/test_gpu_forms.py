"""Forms of the solver kernels that no default launch of these sizes takes,
against those that it does: the same bits."""
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


@pytest.mark.parametrize("qgrad_lanes,residual_lanes", [(0, 1), (4, 1), (0, 4), (4, 8)])
@pytest.mark.parametrize("precision,farfield", [(0, 0), (1, 0), (0, 1)])
def test_tiled_batch_against_gathered_states(lk, precision, farfield, qgrad_lanes, residual_lanes):
    """A batch of 18,432 points (288 tiles: tiled residual) against single states
    of 2,304 and 3,840 points (fewer than 256 tiles: gathered with these lanes), with
    the q-derivative passes tiled and gathered."""
    a = lk.Cloud(cg.ogrid(96, 24, r=1.12, t=0.12))
    b = lk.Cloud(cg.ogrid(128, 30, r=1.1, t=0.10, jitter_p=0.05, seed=3))
    conds = [(0, 0.5, 2.0), (1, 0.63, -1.0), (0, 0.7, 3.0), (1, 0.8, 1.0), (1, 0.4, 0.0), (0, 0.6, 1.0)]
    prm = lk.default_params(cfl=50.0, limiter=1, precision=precision, farfield=farfield,
                            qgrad_lanes=qgrad_lanes, residual_lanes=residual_lanes)
    bat = lk.Batch([a, b], [c[0] for c in conds], [c[1] for c in conds], [c[2] for c in conds], prm)
    for _ in range(3):
        bat.step_timed()
    for k, (ci, m, al) in enumerate(conds):
        st = lk.State([a, b][ci], m, al, prm)
        for _ in range(3):
            st.step(want_res=False)
        assert np.array_equal(bat.get_U(k), st.get_U()), k
        st.close()
    bat.close()


def _shuffled(c, seed):
    """The cloud with its points stored in random order, each point's neighbours in
    the order they had; returns it with the old index of every point."""
    perm = np.random.default_rng(seed).permutation(c.n)
    new = np.empty(c.n, np.int64)
    new[perm] = np.arange(c.n)
    cnt = np.diff(c.nbr_off)[perm]
    off = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    src = np.repeat(c.nbr_off[:-1][perm], cnt) + np.arange(off[-1]) - np.repeat(off[:-1], cnt)
    return cg.Cloud(x=c.x[perm], y=c.y[perm], type=c.type[perm], tx=c.tx[perm], ty=c.ty[perm],
                    nbr_off=off, nbr_idx=new[c.nbr_idx[src]].astype(np.int32)), perm


@pytest.mark.parametrize("kw", [dict(), dict(farfield=1, gamma=1.3)])
@pytest.mark.parametrize("nw,nk", [(160, 40), (160, 126), (640, 260)])
def test_residual_of_shuffled_points_bitwise(lk, nw, nk, kw):
    """A cloud stored row by row (tiled residual: 100 tiles, four threads to a lane;
    320, two; 2,600, one) and the same points in random order, whose tile lists are
    too long (gathered residual): the same bits for every point."""
    c = cg.ogrid(nw, nk, jitter_p=0.03, seed=4)
    s, perm = _shuffled(c, 1)
    prm = lk.default_params(cfl=20.0, limiter=1, qgrad_lanes=4, **kw)
    st = lk.State(lk.Cloud(c), 0.7, 2.0, prm)
    for _ in range(2):
        st.step(want_res=False)
    U = st.get_U()
    st.set_U(U)
    R, _ = st.residual()
    st.close()
    st = lk.State(lk.Cloud(s), 0.7, 2.0, prm)
    st.set_U(np.ascontiguousarray(U[:, perm]))
    assert np.isfinite(R).all() and np.array_equal(st.residual()[0], R[:, perm])
    st.close()


@pytest.mark.parametrize("limiter,inner", [(1, 0), (1, 2), (0, 1)])
@pytest.mark.parametrize("r", [3, 4, 5, 6, 7])
def test_q_derivatives_by_tile_stride(lk, r, limiter, inner):
    """Box clouds with every point within r rows and columns as neighbour: tile
    lists of 220, 288, 364, 448 and 540 points (up to 365, 480 and beyond what a
    tile holds), against the oracle, the suite's bar of 1e-11."""
    c = cg.box(40, 20, wall_bottom=True)
    nx, ny = c.nw, c.nk
    off, idx = [0], []
    for p in range(c.n):
        j, k = p % nx, p // nx
        idx += [q * nx + i for q in range(max(0, k - r), min(ny, k + r + 1))
                for i in range(max(0, j - r), min(nx, j + r + 1)) if q * nx + i != p]
        off.append(len(idx))
    c.nbr_off, c.nbr_idx = np.array(off, np.int32), np.array(idx, np.int32)
    kw = dict(cfl=5.0, inner_iters=inner, limiter=limiter, limiter_k=5.0)
    o = O.Oracle(c, mach=0.4, aoa_deg=5.0, **kw)
    bump = np.stack([np.sin(2 * c.x + c.y), np.cos(c.x - 2 * c.y), np.sin(c.x * c.y), np.cos(3 * c.x)])
    U = o.free_stream() * (1.0 + 0.05 * bump)
    U[2, c.type == 0] = 0.0
    st = lk.State(lk.Cloud(c), 0.4, 5.0, lk.default_params(**kw))
    st.set_U(U)
    got = (*st.q_derivatives(), st.residual()[0])
    want = (*o.q_derivatives(O.q_from_U(U)), o.residual(U)[0])
    errs = [max(np.abs(a[v] - b[v]).max() / np.abs(b[v]).max() for v in range(4))
            for a, b in zip(got, want)]
    assert np.isfinite(errs).all() and max(errs) < 1e-11, errs
    st.close()

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


@pytest.mark.parametrize("kw", [dict(), dict(precision=1), dict(jvp_mode=1), dict(farfield=1)])
def test_sweeps_of_8_and_16_lanes_agree_bitwise(lk, kw):
    """Lists of at most 32 entries: sixteen lanes add in the order of eight."""
    gc = lk.Cloud(cg.ogrid(96, 24, r=1.12))
    got = []
    for lanes in (8, 16):
        st = lk.State(gc, 0.6, 2.0, lk.default_params(cfl=50.0, limiter=1, sweep_lanes=lanes, **kw))
        for _ in range(3):
            st.step(want_res=False)
        got.append((st.get_dU(), st.get_U()))
        st.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


def _ring(cloud, r):
    """The box cloud with every point within r rows and columns as neighbour."""
    nx, ny = cloud.nw, cloud.nk
    off, idx = [0], []
    for p in range(cloud.n):
        j, k = p % nx, p // nx
        idx += [q * nx + i for q in range(max(0, k - r), min(ny, k + r + 1))
                for i in range(max(0, j - r), min(nx, j + r + 1)) if q * nx + i != p]
        off.append(len(idx))
    cloud.nbr_off, cloud.nbr_idx = np.array(off, np.int32), np.array(idx, np.int32)
    return cloud


@pytest.mark.parametrize("lanes", [0, 1, 2, 4, 8, 16])
def test_sweeps_with_long_lists(lk, lanes):
    """Up to 80 neighbours a point (lists beyond 32 entries) at every lane
    count, wall and outer points among them: one increment against the oracle,
    the suite's bar of 1e-11."""
    cloud = _ring(cg.box(15, 14, wall_bottom=True), 4)
    kw = dict(cfl=5.0, inner_iters=0)
    o = O.Oracle(cloud, mach=0.4, aoa_deg=5.0, **kw)
    rng = np.random.default_rng(5)
    U = o.free_stream() * (1.0 + 0.01 * rng.uniform(-1, 1, (4, cloud.n)))
    U[2, cloud.type == 0] = 0.0
    _, _, dUo, _ = o.iteration(U)
    st = lk.State(lk.Cloud(cloud), 0.4, 5.0, lk.default_params(sweep_lanes=lanes, **kw))
    st.set_U(U)
    st.step()
    dU = st.get_dU()
    e = max(np.abs(dU[v] - dUo[v]).max() / np.abs(dUo[v]).max() for v in range(4))
    print(f"long lists, {lanes} lanes: {e:.2e}")
    assert np.isfinite(e) and e < 1e-11


@pytest.mark.parametrize("r,inner", [(1, 0), (2, 1), (3, 2), (4, 1), (4, 0)])
def test_q_derivatives_by_list_length(lk, r, inner):
    """Stencils of 8 to 80 neighbours on a 40 x 20 box: tile lists below and
    above the staged arrays' usual stride (160), entries beyond the 32 whose
    positions a point's lanes hold; q-derivatives and the limited residual
    against the oracle, the suite's bar of 1e-11."""
    cloud = _ring(cg.box(40, 20, wall_bottom=True), r)
    kw = dict(cfl=5.0, inner_iters=inner, limiter=1, limiter_k=5.0)
    o = O.Oracle(cloud, mach=0.4, aoa_deg=5.0, **kw)
    rng = np.random.default_rng(6)
    x, y = cloud.x, cloud.y
    bump = np.stack([np.sin(2 * x + y), np.cos(x - 2 * y), np.sin(x * y), np.cos(3 * x)])
    U = o.free_stream() * (1.0 + 0.05 * bump + 0.001 * rng.uniform(-1, 1, (4, cloud.n)))
    U[2, cloud.type == 0] = 0.0
    st = lk.State(lk.Cloud(cloud), 0.4, 5.0, lk.default_params(**kw))
    st.set_U(U)
    R, _ = st.residual()
    qx, qy = st.q_derivatives()
    ox, oy = o.q_derivatives(O.q_from_U(U))
    Ro, _ = o.residual(U)
    errs = [max(np.abs(a[v] - b[v]).max() / np.abs(b[v]).max() for v in range(4))
            for a, b in ((qx, ox), (qy, oy), (R, Ro))]
    print(f"radius {r}, {inner} inner: {errs}")
    assert np.isfinite(errs).all() and max(errs) < 1e-11


def test_features_nearest_wall(lk):
    """The nearest-wall search by runs of wall points: a wall of many runs with
    a short last one (330 points), clouds without a wall, and a batch of
    25-point clouds whose conditions share wavefronts, against the brute force
    of the oracle (float32 features: 1e-6)."""
    from oracle import mlp as OM
    c = cg.ogrid(330, 24, jitter_p=0.05, seed=2)
    st = lk.State(lk.Cloud(c), 0.7, 1.0, lk.default_params())
    X = st.features().cpu().numpy()
    assert np.abs(X - OM.features(c.x, c.y, c.type, 0.7, 1.0)).max() <= 1e-6
    st.close()
    clouds = [cg.box(5, 5, wall_bottom=True), cg.box(5, 5), c]
    which = [0, 1, 0, 1, 0, 2, 1]
    mach = [0.3 + 0.05 * k for k in range(7)]
    b = lk.Batch([lk.Cloud(x) for x in clouds], which, mach, [0.0] * 7, lk.default_params())
    X = b.features().cpu().numpy()
    o = 0
    for k, w in enumerate(which):
        ref = OM.features(clouds[w].x, clouds[w].y, clouds[w].type, mach[k], 0.0)
        assert np.abs(X[o:o + clouds[w].n] - ref).max() <= 1e-6, k
        o += clouds[w].n
    b.close()


@pytest.mark.parametrize("m", [1, 15, 16, 17, 32, 33, 8193, 16417])
def test_mlp_rows_at_tile_edges(lk, m):
    """Forward (16 rows a wave, 128 a block) and gradient (32 rows a turn, at
    most 256 blocks: 8,193 rows are the first second turn) against the oracle.
    One activation rounded to bfloat16 the other way moves a gradient by about
    2^-8 / sqrt(128) = 3.5e-4 of its norm; few are: 2e-3."""
    import torch
    from oracle import mlp as OM
    rng = np.random.default_rng(m)
    th = np.concatenate([rng.uniform(-1, 1, int(np.prod(s))) * (0.15 if len(s) > 1 else 0.1)
                         for _, s in OM.SHAPES]).astype(np.float32)
    X = rng.uniform(-1, 1, (m, 5)).astype(np.float32)
    T = (0.3 * np.sin(np.pi * X[:, :4]) * X[:, 4:5]).astype(np.float32)
    dX, dT = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    net = lk.MLP(max_rows=m)
    net.set_params(th)
    Y = net.forward(dX).cpu().numpy()
    loss, g = net.gradient(dX, dT)
    # rows do not depend on their place: the same bits for the rows alone
    cut = m // 2
    assert np.array_equal(Y, np.concatenate([net.forward(dX[k]).cpu().numpy()
                                             for k in (slice(0, cut), slice(cut, m))]))
    net.close()
    th, X, T = th.astype(np.float64), X.astype(np.float64), T.astype(np.float64)
    ref, _ = OM.forward(th, X)
    err = np.abs(Y - ref) / np.abs(ref).max()
    assert np.quantile(err, 0.99) <= 1e-3 and err.max() <= 2e-2, err.max()
    rl, rg = OM.loss_and_grad(th, X, T)
    assert abs(loss - rl) <= 1e-3 * rl
    o = 0
    for name, shape in OM.SHAPES:
        k = int(np.prod(shape))
        assert np.linalg.norm(g[o:o + k] - rg[o:o + k]) <= 2e-3 * np.linalg.norm(rg[o:o + k]), name
        o += k


@pytest.mark.parametrize("nx,ny", [(5, 5), (4681, 7), (2048, 16), (331, 99), (5243, 25)])
def test_host_fields_by_chunks(lk, nx, ny):
    """Fields to and from host arrays cross in chunks of 32,768 points through
    three slots (25, 32,767, 32,768, 32,769 and 4 x 32,768 + 3 points): every
    value arrives, the same as by the device route."""
    import torch
    c = cg.box(nx, ny)
    U = np.empty((4, c.n))
    U[0] = 1.0 + 1e-3 * np.arange(c.n) / c.n
    U[1], U[2] = 0.3, -0.1 * np.arange(c.n) / c.n
    U[3] = 2.5 + 1e-4 * np.arange(c.n)[::-1] / c.n
    st = lk.State(lk.Cloud(c), 0.5, 1.0, lk.default_params())
    st.set_U(U)
    assert np.array_equal(st.get_U(), U)
    st.set_U(torch.from_numpy(U + 1e-3).cuda())
    assert np.array_equal(st.get_U(), st.get_U(device=True).cpu().numpy())
    st.close()
    small = lk.Cloud(cg.box(5, 5))
    b = lk.Batch([small, lk.Cloud(c)], [0, 1, 0], [0.5] * 3, [0.0] * 3, lk.default_params())
    b.set_U(1, U)
    assert np.array_equal(b.get_U(1), U)
    assert np.array_equal(b.get_U(0), b.get_U(2))
    b.close()


@pytest.mark.parametrize("nw,nk", [(20, 6), (160, 40), (160, 110)])
@pytest.mark.parametrize("kw", [dict(), dict(precision=1), dict(farfield=1, gamma=1.3)])
def test_residual_threads_per_lane_bitwise(lk, nw, nk, kw):
    """Four threads to a lane (2 and 100 tiles), two (275 and more) and the
    forms that two asked-for lanes take (gathered, tiled): the same bits."""
    c = lk.Cloud(cg.ogrid(nw, nk, jitter_p=0.03, seed=4))
    out = []
    for lanes in (0, 2):
        st = lk.State(c, 0.7, 2.0, lk.default_params(cfl=20.0, limiter=1, residual_lanes=lanes, **kw))
        for _ in range(3):
            st.step(want_res=False)
        out.append((st.residual(), st.get_U()))
        st.close()
    (a, ra), ua = out[0]
    (b, rb), ub = out[1]
    assert np.isfinite(a).all() and ra == rb
    assert np.array_equal(a, b) and np.array_equal(ua, ub)


@pytest.mark.parametrize("nw", [64, 2048, 2100])
def test_features_by_wall_runs(lk, nw):
    """Walls of 2, 64 and 66 runs of 32 points (a wavefront bounds 64 runs at a
    time), points near and far, a last wavefront that is not full."""
    from oracle import mlp as OM
    c = cg.ogrid(nw, 7, r=2.5, jitter_p=0.03, seed=5)
    st = lk.State(lk.Cloud(c), 0.7, 1.0, lk.default_params())
    X = st.features().cpu().numpy()
    assert np.abs(X - OM.features(c.x, c.y, c.type, 0.7, 1.0)).max() <= 1e-6
    st.close()


@pytest.mark.parametrize("kw", [dict(), dict(precision=1), dict(jvp_mode=1), dict(farfield=1),
                                dict(variant=1)])
@pytest.mark.parametrize("nw,nk", [(16, 5), (160, 40), (160, 126)])
def test_sweep_lanes_of_small_clouds_bitwise(lk, nw, nk, kw):
    """Thirty-two lanes per point (80 and 6,400 points), sixteen (20,160) and the
    eight that are asked for: the same bits."""
    c = lk.Cloud(cg.ogrid(nw, nk, jitter_p=0.03, seed=6))
    out = []
    for lanes in (0, 8):
        st = lk.State(c, 0.6, 2.0, lk.default_params(cfl=20.0, limiter=1, sweep_lanes=lanes, **kw))
        for _ in range(3):
            st.step(want_res=False)
        out.append((st.get_U(), st.get_dU()))
        st.close()
    assert np.isfinite(out[0][0]).all() and np.any(out[0][1])
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])

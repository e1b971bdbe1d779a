"""Tiles whose every cell holds one state are advanced without evaluating a
face: bit for bit the oracle's result, on uniform states, on states with one
cell that differs (in any component, down to the sign of a zero; at any
distance from tile edges), with every boundary kind, and on uniform states
outside the bounds within which the shortcut is taken."""
import numpy as np
import pytest

import oracle
from paper_1707_00592_amd import workloads as wl
from test_gpu_division_ranges import _dev, _same_bits

pytestmark = pytest.mark.gpu

SHAPES = [(5,), (520,), (47, 35), (30, 32), (64, 18, 16), (33, 7, 31)]
# rho, u, p, gamma, Pinf: water and air at rest and moving, and states the
# shortcut refuses (hypersonic, near vacuum, tension close to the stiffness)
STATES = [(1000.0, 0.0, 1e5, 4.4, 6e8), (1.0, 300.0, 1e5, 1.4, 0.0), (1.0, -30.0, 1e5, 1.4, -0.0),
          (1.0, 1e5, 1e2, 1.4, 0.0), (1e-5, 0.0, 1e5, 1.4, 0.0), (1000.0, 1.0, -5.9e8, 4.4, 6e8)]


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


def _uniform(shape, w, seed):
    rs = np.random.default_rng(seed)
    n = int(np.prod(shape))
    vel = [np.full(n, w[1] * f) for f in (1.0, 0.0, -0.5)[:len(shape)]]
    if rs.random() < 0.5:
        vel[-1] = -0.0 * np.ones(n)
    return wl.prim_to_cons(np.full(n, w[0]), vel, w[2], w[3], w[4])


def _step_and_rhs(lib, ctx, U, shape, bc, precision=0):
    dx = tuple(1.0 / m for m in shape)
    ig = lib.make_grid(shape, dx, bc, bc)
    o = lib.make_opts(precision=precision)
    st = lib.new_stats()
    rhs = ctx.rhs(_dev(U), ig, o, stats=st).cpu().numpy()
    V = _dev(U)
    import torch
    dt = torch.zeros(1, dtype=torch.float64, device="cuda")
    for _ in range(2):
        ctx.rk3_step(V, ig, o, dt, st)
    return rhs, V.cpu().numpy(), lib.read_stats(st)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("which", range(len(STATES)))
def test_uniform_and_one_cell_off(lib, ctx, shape, bc, which):
    rs = np.random.default_rng(which)
    d = len(shape)
    og = oracle.make_grid(shape, tuple(1.0 / m for m in shape), (bc,) * d, (bc,) * d)
    for k in range(6):
        U = _uniform(shape, STATES[which], k)
        if k:  # one cell, one component: a small change or the other zero
            c, cell = int(rs.integers(0, 4 + d)), int(rs.integers(0, U.shape[1]))
            U[c, cell] = -U[c, cell] if U[c, cell] == 0 else U[c, cell] * (1 + 1e-9)
        rhs, V, st = _step_and_rhs(lib, ctx, U, shape, (bc,) * d)
        ref, s0 = oracle.rhs(U, og, oracle.make_opts())
        assert _same_bits(rhs, ref), (shape, bc, which, k)
        W = U
        for _ in range(2):
            h = oracle.cfl_dt(W, og, oracle.make_opts())
            W, s1 = oracle.rk3_step(W, og, h, oracle.make_opts())
        if st.status == 0:
            assert s1 == 0 and _same_bits(V, W), (shape, bc, which, k)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bc", [0, 1, 2])
def test_float_form_keeps_uniform_states(lib, ctx, shape, bc):
    """The float form: a uniform state has dU/dt of signed zeros equal to the
    FP64 form's (every difference is x - x)."""
    d = len(shape)
    for which in (0, 1):
        U = _uniform(shape, STATES[which], which)
        if bc != 2 or STATES[which][1] == 0.0:
            rhs64, _, _ = _step_and_rhs(lib, ctx, U, shape, (bc,) * d)
            rhs32, _, _ = _step_and_rhs(lib, ctx, U, shape, (bc,) * d, precision=1)
            assert _same_bits(rhs32, rhs64)


def test_batch_of_uniform_and_mixed_tubes(lib, ctx):
    """Uneven tubes, uniform ones among tubes with a jump: the oracle's bits
    problem by problem."""
    import torch
    rs = np.random.default_rng(4)
    sizes = [1, 2, 62, 63, 64, 255, 256, 700, 1024, 90]
    parts, dxs = [], []
    for k, n in enumerate(sizes):
        U = _uniform((n,), STATES[k % 2], k)
        if k % 3 == 2:
            U[:, rs.integers(0, n):] = _uniform((1,), STATES[0], 0)
        parts.append(U)
        dxs.append(1.0 / n)
    off = np.concatenate([[0], np.cumsum(sizes)])
    plan = ctx.batch_plan(off, dxs, 0, 0)
    V = _dev(np.concatenate(parts, axis=1))
    dt = torch.zeros(len(sizes), dtype=torch.float64, device="cuda")
    o = lib.make_opts()
    plan.step(V, o, dt, 3)
    got = V.cpu().numpy()
    for k, n in enumerate(sizes):
        og = oracle.make_grid((n,), (dxs[k],), (0,), (0,))
        W = parts[k]
        for _ in range(3):
            h = oracle.cfl_dt(W, og, oracle.make_opts())
            W, _ = oracle.rk3_step(W, og, h, oracle.make_opts())
        assert _same_bits(got[:, off[k]:off[k + 1]], W), n


def _same_or_nan(a, b):
    """Equal bits, NaN where the other is NaN."""
    return np.array_equal(np.isnan(a), np.isnan(b)) and _same_bits(np.where(np.isnan(a), 0.0, a),
                                                                   np.where(np.isnan(b), 0.0, b))


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("mood", [False, True])
@pytest.mark.parametrize("weights", [oracle.W_MODIFIED, oracle.W_BASIC])
def test_epsilon_zero_is_not_skipped(lib, ctx, shape, mood, weights):
    """epsilon = 0: a constant stencil's weights are 0/0, so a uniform tile's
    derivative is NaN without the cascade and each of its face sides falls
    back with it, as everywhere else."""
    d = len(shape)
    dx = tuple(1.0 / m for m in shape)
    ig, og = lib.make_grid(shape, dx, 0, 0), oracle.make_grid(shape, dx, (0,) * d, (0,) * d)
    o = lib.make_opts(weights=weights, mood=mood, eps=0.0)
    oo = oracle.make_opts(weights=weights, mood=mood, eps=0.0)
    for k in range(2):
        U = _uniform(shape, STATES[k], k)
        if k:  # mixed and uniform tiles side by side
            U[:, U.shape[1] // 2] *= 1.001
        st = lib.new_stats()
        got = ctx.rhs(_dev(U), ig, o, stats=st).cpu().numpy()
        ref, so = oracle.rhs(U, og, oo)
        assert np.isnan(ref).any() != mood and _same_or_nan(got, ref), k
        s = lib.read_stats(st)
        assert (list(s.o3), list(s.o1)) == (list(so.o3), list(so.o1)) and any(so.o1) == mood


@pytest.mark.parametrize("bc", [0, 1])
def test_epsilon_zero_batch(lib, ctx, bc):
    """The same in a batch, whole steps and stage launches."""
    import torch
    sizes = [40, 700, 255]
    off = np.concatenate([[0], np.cumsum(sizes)])
    U = _uniform((int(off[-1]),), STATES[0], 0)
    dxs = np.array([1.0 / n for n in sizes])
    ref, dtr, so, s, ps = oracle.batch_step(U, off, dxs, oracle.make_opts(eps=0.0), bc_lo=bc,
                                            bc_hi=bc, pstatus=np.zeros(3, np.intc))
    plan, V, st = ctx.batch_plan(off, dxs, bc, bc), _dev(U), lib.new_stats()
    dt = torch.zeros(3, dtype=torch.float64, device="cuda")
    plan.step(V, lib.make_opts(eps=0.0), dt, 1, st)
    assert list(plan.status.cpu().numpy()) == list(ps) == [0, 0, 0]
    assert _same_bits(V.cpu().numpy(), ref)
    got = lib.read_stats(st)
    assert (got.o3[0], got.o1[0]) == (so.o3[0], so.o1[0]) and so.o1[0] > 0


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("which", range(len(STATES)))
def test_status_and_steps_match_the_oracle(lib, ctx, shape, which):
    """Step by step, the status first: a failure that only one side latches is
    an error, not a reason to compare nothing."""
    import torch
    d = len(shape)
    dx = tuple(1.0 / m for m in shape)
    og, ig = oracle.make_grid(shape, dx, (0,) * d, (0,) * d), lib.make_grid(shape, dx, 0, 0)
    for k in range(2):
        W = _uniform(shape, STATES[which], k)
        if k:
            W[:, W.shape[1] // 3] *= 1 + 1e-9
        U, st = _dev(W), lib.new_stats()
        dt = torch.zeros(1, dtype=torch.float64, device="cuda")
        for step in range(3):
            ctx.rk3_step(U, ig, lib.make_opts(), dt, st)
            W, s = oracle.rk3_step(W, og, oracle.cfl_dt(W, og, oracle.make_opts()), oracle.make_opts())
            assert lib.read_stats(st).status == s, (k, step)
            if s != 0:
                break
            assert _same_bits(U.cpu().numpy(), W), (k, step)


@pytest.mark.parametrize("shape", [(300, 409), (301, 417), (420, 410)])
@pytest.mark.parametrize("mood", [1, 2])
def test_float_form_on_both_sides_of_the_tile_count(lib, ctx, shape, mood):
    """520 and 480, 567 and 504, 728 and 672 tiles: the float form tells uniform
    tiles apart beyond 512.  A uniform state keeps the FP64 form's signed zeros,
    one with a pressure bump its derivative within 1e-3 (relative L1: fluxes are
    rounded to float, 6e-8, and differ by percents across the bump) and zeros
    away from it."""
    for ny in (shape[1], shape[1] - 40):
        n = (shape[0], ny)
        ig = lib.make_grid(n, (0.01, 0.01), 0, 0)
        U = _uniform(n, STATES[1], 1)
        a, b = (ctx.rhs(_dev(U), ig, lib.make_opts(precision=p, mood=mood)).cpu().numpy()
                for p in (0, 1))
        assert _same_bits(a, b)
        x, y = np.meshgrid(np.arange(n[0]), np.arange(n[1]))
        r2 = ((x - 100) ** 2 + (y - 120) ** 2).ravel()
        U[3] *= 1 + 0.1 * np.maximum(0, 1 - r2 / 400.0)
        a, b = (ctx.rhs(_dev(U), ig, lib.make_opts(precision=p, mood=mood)).cpu().numpy()
                for p in (0, 1))
        assert np.abs(b - a).sum() <= 1e-3 * np.abs(a).sum()
        assert (b[:, r2 > 26 ** 2] == 0).all() and (b[:, r2 < 16 ** 2] != 0).any()

"""The MOOD cascade where it acts: states of wild cells (every wave holds
sides that fail), alone and with cells outside the range of the unscaled
divisions among them.  The oracle's derivative, bit for bit, and its MOOD
counts, on lines of one launch and longer ones, in 2D with the cascade in its
wave and gathered, in 3D, and in batches with whole steps and stage launches."""
import numpy as np
import pytest

import oracle
from paper_1707_00592_amd import workloads as wl
from test_gpu_division_ranges import _dev, _same_bits

pytestmark = pytest.mark.gpu

FORMS = [oracle.W_MODIFIED, oracle.W_BASIC, oracle.W_CUTOFF]
SHAPES = [(64,), (300,), (700,), (47, 35), (130, 70), (37, 18, 19)]


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


def _wild(shape, share, far, seed):
    """Water at rest with `share` of its cells random two-phase states and
    `far` of them thinner than 2^-20."""
    rs = np.random.default_rng(seed)
    n = int(np.prod(shape))
    wild = rs.random(n) < share
    gas = wild & (rs.random(n) < 0.5)
    rho = np.where(gas, 1.0, 1000.0) * np.where(wild, rs.uniform(0.5, 2, n), 1.0)
    rho = np.where(rs.random(n) < far, 1e-7, rho)
    vel = [np.where(wild, rs.uniform(-2000, 2000, n), 0.0) for _ in shape]
    p = np.where(wild, 10 ** rs.uniform(4, 9.5, n), 1e5)
    return wl.prim_to_cons(rho, vel, p, np.where(gas, 1.4, 4.4), np.where(gas, 0.0, 6e8))


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("weights", FORMS)
@pytest.mark.parametrize("share,far", [(1.0, 0.0), (0.3, 0.0), (1.0, 0.02)])
def test_derivative_and_counts(lib, ctx, shape, weights, share, far):
    d = len(shape)
    dx = tuple(1.0 / m for m in shape)
    og = oracle.make_grid(shape, dx, (0,) * d, (2,) * d)
    ig = lib.make_grid(shape, dx, 0, 2)
    U = _wild(shape, share, far, d)
    ref, so = oracle.rhs(U, og, oracle.make_opts(weights=weights))
    assert sum(so.o3) + sum(so.o1) > 0
    for mood in (lib.MOOD_ON, lib.MOOD_GATHER) if d == 2 else (lib.MOOD_ON,):
        st = lib.new_stats()
        got = ctx.rhs(_dev(U), ig, lib.make_opts(weights=weights, mood=mood), stats=st)
        s = lib.read_stats(st)
        assert _same_bits(got.cpu().numpy(), ref), mood
        assert (list(s.o3), list(s.o1)) == (list(so.o3), list(so.o1)), mood


@pytest.mark.parametrize("n", [64, 255, 256, 511, 512])
@pytest.mark.parametrize("weights", FORMS)
def test_a_line_s_step_and_counts(lib, ctx, n, weights):
    import torch
    U0 = _wild((n,), 1.0, 0.0, n)
    ig, og = lib.make_grid((n,), (1.0 / n,), 0, 0), oracle.make_grid((n,), (1.0 / n,), (0,), (0,))
    oo, so = oracle.make_opts(weights=weights, cfl=0.005), oracle.Stats()
    h = oracle.cfl_dt(U0, og, oo)
    W, status = oracle.rk3_step(U0, og, h, oo, so)
    U, st = _dev(U0), lib.new_stats()
    dt = torch.zeros(1, dtype=torch.float64, device="cuda")
    ctx.rk3_step(U, ig, lib.make_opts(weights=weights, cfl=0.005), dt, st)
    s = lib.read_stats(st)
    assert s.status == status and float(dt.item()) == h
    if status == 0:
        assert _same_bits(U.cpu().numpy(), W)
        assert (s.o3[0], s.o1[0]) == (so.o3[0], so.o1[0]) and so.o3[0] + so.o1[0] > 0


@pytest.mark.parametrize("bc", [(0, 0), (1, 1)])
@pytest.mark.parametrize("weights", FORMS)
def test_batch_step_and_counts(lib, ctx, bc, weights):
    import torch
    sizes = [3, 40, 243, 256, 700]
    off = np.concatenate([[0], np.cumsum(sizes)])
    dxs = np.array([1.0 / n for n in sizes])
    U0 = np.concatenate([_wild((n,), 1.0, 0.0, n) for n in sizes], axis=1)
    ref, dtr, so, _, ps = oracle.batch_step(U0, off, dxs, oracle.make_opts(weights=weights, cfl=0.005),
                                            bc_lo=bc[0], bc_hi=bc[1],
                                            pstatus=np.zeros(len(sizes), np.intc))
    plan, U, st = ctx.batch_plan(off, dxs, *bc), _dev(U0), lib.new_stats()
    dt = torch.zeros(len(sizes), dtype=torch.float64, device="cuda")
    plan.step(U, lib.make_opts(weights=weights, cfl=0.005), dt, 1, st)
    got, s = U.cpu().numpy(), lib.read_stats(st)
    assert list(plan.status.cpu().numpy()) == list(ps)
    for k in range(len(sizes)):
        if ps[k] == 0:
            assert _same_bits(got[:, off[k]:off[k + 1]], ref[:, off[k]:off[k + 1]]), sizes[k]
    if not any(ps):
        assert (s.o3[0], s.o1[0]) == (so.o3[0], so.o1[0]) and so.o3[0] + so.o1[0] > 0

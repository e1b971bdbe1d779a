"""Batches at every lane count, chosen by hand instead of by the autotuner's
timing: whole steps at the edges of their tiles, and the stage launches of
plans with a periodic end with several tiles a tube, uniform tubes among mixed
ones and more tiles than workgroups.  FP64: the oracle's bits, time steps and
MOOD counts; float form within 2e-4 (relative L1) of the oracle.  Fixed time
steps, and a tube that is frozen before the call, likewise."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_1707_00592_amd import workloads as wl
from test_gpu_batch_whole_steps import _tubes
from test_gpu_division_ranges import _dev

pytestmark = pytest.mark.gpu

LANES = [64, 128, 256]


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


def _plan(lib, ctx, b, bc, lanes):
    plan = ctx.batch_plan(b["offsets"], b["dx"], *bc)
    f = lib.load().isweno_test_batch_lanes
    f.argtypes, f.restype = [C.c_void_p, C.c_int32], C.c_int
    lib.check(f(plan._h, lanes))
    return plan


def _compare(lib, plan, b, bc, weights, precision=0, nsteps=2, cfl=0.4, dt0=None, frozen=()):
    import torch
    nprob = len(b["dx"])
    ps0 = np.zeros(nprob, np.intc)
    ps0[list(frozen)] = oracle.ERR_NONPHYSICAL
    ref, dtr, st, _, ps = oracle.batch_step(b["U"], b["offsets"], b["dx"],
                                            oracle.make_opts(weights=weights, cfl=cfl), dt=dt0,
                                            nsteps=nsteps, bc_lo=bc[0], bc_hi=bc[1], pstatus=ps0)
    U = _dev(b["U"])
    dt = torch.zeros(nprob, dtype=torch.float64, device="cuda") if dt0 is None else _dev(dt0)
    stats, status = lib.new_stats(), _dev(ps0.astype(np.int32))
    plan.step(U, lib.make_opts(weights=weights, precision=precision, cfl=cfl), dt, nsteps, stats,
              status)
    got, off = U.cpu().numpy(), b["offsets"]
    if precision:
        assert (status.cpu().numpy() == ps).all()
        assert np.abs(got - ref).sum() <= 2e-4 * np.abs(ref).sum()
        return
    assert (status.cpu().numpy() == ps).all()
    for k in range(nprob):
        sl = slice(off[k], off[k + 1])
        if ps[k] == 0 or k in frozen:
            np.testing.assert_array_equal(got[:, sl], (b["U"] if k in frozen else ref)[:, sl])
            if k not in frozen:
                assert float(dt[k].item()) == dtr[k]
    if not any(ps):
        s = lib.read_stats(stats)
        assert (s.o3[0], s.o1[0]) == (st.o3[0], st.o1[0])


@pytest.mark.parametrize("lanes", LANES)
@pytest.mark.parametrize("bc", [(0, 0), (2, 2), (2, 0)])
@pytest.mark.parametrize("weights", [oracle.W_MODIFIED, oracle.W_CUTOFF])
def test_whole_steps(lib, ctx, lanes, bc, weights):
    tile = lanes - 13
    sizes = [3, 9, 10, tile - 1, *range(tile, tile + 11), 2 * tile, 2 * tile + 1, 3 * tile + 8]
    b = _tubes(sizes, lanes)
    plan = _plan(lib, ctx, b, bc, lanes)
    _compare(lib, plan, b, bc, weights)
    dt0 = 0.1 * b["dx"] / 3000.0
    _compare(lib, plan, b, bc, weights, cfl=0.0, dt0=dt0, frozen=(3, len(sizes) - 1))
    if bc == (0, 0):
        _compare(lib, plan, b, bc, weights, precision=1)


@pytest.mark.parametrize("lanes", LANES)
@pytest.mark.parametrize("bc", [(1, 1), (2, 1), (1, 0)])
@pytest.mark.parametrize("weights,precision", [(oracle.W_MODIFIED, 0), (oracle.W_CUTOFF, 0),
                                               (oracle.W_MODIFIED, 1), (oracle.W_CUTOFF, 1)])
def test_stage_launches(lib, ctx, lanes, bc, weights, precision):
    """More tiles than the 4 workgroups a compute unit of the default."""
    import torch
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    tile = lanes - 1
    rs = np.random.default_rng(lanes)
    sizes, tiles = [3, tile, tile + 1, 2 * tile + 3], 0
    while tiles <= 4 * ncu + 5:
        sizes.append(int(rs.integers(tile // 2, 4 * tile)))
        tiles = sum(-(-n // tile) for n in sizes)
    states, x0s = [], []
    for k in range(len(sizes)):  # every third tube uniform, the others a mild jump
        left = (1000.0, 3.0, 1e5, *wl.WATER)
        right = left if k % 3 == 0 else (1.2, 3.0, 2e5, *wl.AIR) if k % 3 == 1 else \
            (990.0, -2.0, 4e6, *wl.WATER)
        states.append((left, right))
        x0s.append(0.2 + 0.6 * rs.random())
    b = wl.batch_from_states(sizes, states, x0s)
    _compare(lib, _plan(lib, ctx, b, bc, lanes), b, bc, weights, precision=precision, nsteps=1)

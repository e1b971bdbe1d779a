"""Whole steps of batched tubes (one launch per step): problem lengths at the
edges of its tiles and of the cells a tile reads beyond its ends, for each
number of lanes (the regime's lengths make it the likely choice of the
autotuner; the default is the largest), every non-periodic boundary kind,
several steps in place.  The oracle's bits, time steps and MOOD counts."""
import numpy as np
import pytest

import oracle
from paper_1707_00592_amd import workloads as wl
from test_gpu_division_ranges import _dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


def _tubes(sizes, seed):
    rs = np.random.default_rng(seed)
    states, x0s = [], []
    for _ in sizes:
        side = []
        for _s in range(2):
            water = rs.random() < 0.5
            side.append((10 ** rs.uniform(2.5, 3) if water else 10 ** rs.uniform(0, 1.5),
                         rs.uniform(-20, 20), 10 ** rs.uniform(5, 8 if water else 6.5),
                         *(wl.WATER if water else wl.AIR)))
        states.append(tuple(side))
        x0s.append(rs.choice([rs.uniform(0.05, 0.95), 0.01, 0.99]))
    return wl.batch_from_states(sizes, states, x0s)


@pytest.mark.parametrize("tile", [51, 115, 243])
@pytest.mark.parametrize("bc", [(0, 0), (2, 2), (0, 2), (2, 0)])
@pytest.mark.parametrize("tuned", [False, True])
def test_tile_edges(lib, ctx, tile, bc, tuned):
    import torch
    sizes = [3, 4, 8, 9, 10, tile - 1, tile, *range(tile + 1, tile + 13), 2 * tile - 1, 2 * tile,
             2 * tile + 1, 2 * tile + 8, 3 * tile + 9]
    if not any(bc):
        sizes += [1, 2]
    b = _tubes(sizes, tile)
    o = lib.make_opts(mood=True, cfl=0.4)
    oo = oracle.make_opts(mood=True, cfl=0.4)
    ref, dtr, st, _, ps = oracle.batch_step(b["U"], b["offsets"], b["dx"], oo, nsteps=4, bc_lo=bc[0],
                                            bc_hi=bc[1], pstatus=np.zeros(len(sizes), np.intc))
    plan = ctx.batch_plan(b["offsets"], b["dx"], *bc)
    U = _dev(b["U"])
    chosen = plan.autotune(U, o) if tuned else 255
    dt = torch.zeros(len(sizes), dtype=torch.float64, device="cuda")
    stats = lib.new_stats()
    plan.step(U, o, dt, 1, stats)
    plan.step(U, o, dt, 3, stats)
    got, s = U.cpu().numpy(), lib.read_stats(stats)
    print(f"[whole steps] tile {tile} bc {bc}: lanes {chosen + 1}, frozen {sum(ps != 0)}", flush=True)
    assert list(plan.status.cpu().numpy()) == list(ps)
    for k, n in enumerate(sizes):
        if ps[k] == 0:
            sl = slice(b["offsets"][k], b["offsets"][k + 1])
            np.testing.assert_array_equal(got[:, sl], ref[:, sl], err_msg=f"n = {n}")
            assert float(dt[k].item()) == dtr[k]
    if not any(ps):
        assert (s.o3[0], s.o1[0]) == (st.o3[0], st.o1[0])


@pytest.mark.parametrize("weights", [oracle.W_BASIC, oracle.W_CUTOFF])
def test_weights_and_fixed_time_step(lib, ctx, weights):
    sizes = [5, 243, 244, 250, 252, 500]
    b = _tubes(sizes, 9)
    dt0 = 0.1 * b["dx"] / 3000.0
    ref, *_ = oracle.batch_step(b["U"], b["offsets"], b["dx"],
                                oracle.make_opts(weights=weights, mood=False, cfl=0.0), dt=dt0,
                                nsteps=2)
    plan = ctx.batch_plan(b["offsets"], b["dx"])
    U = _dev(b["U"])
    plan.step(U, lib.make_opts(weights=weights, mood=False, cfl=0.0), _dev(dt0), 2)
    np.testing.assert_array_equal(U.cpu().numpy(), ref)

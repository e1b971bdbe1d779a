"""Cells and halos of tiles at and near the ends of lines: grids whose lines
are shorter than the three halo cells, end within three cells of a tile's
edge or hold exactly a tile, with every boundary kind at either end of each
axis, against the oracle bit for bit (right-hand side and two steps)."""
import numpy as np
import pytest

import oracle
from paper_1707_00592_amd import workloads as wl
from test_gpu_division_ranges import _dev, _same_bits

pytestmark = pytest.mark.gpu

# 1D lines of more than 511 cells take the sweeps; the 2D tile is 15 x 16, the
# 3D tiles 31 along x and 15 along y and z
SHAPES = [(527,), (528,), (558,), (1, 1), (1, 17), (2, 3), (15, 16), (16, 17), (18, 19), (33, 35),
          (1, 1, 1), (2, 1, 31), (31, 15, 15), (32, 16, 18), (34, 33, 2), (65, 3, 17)]


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("ends", [(0, 0), (1, 1), (2, 2), (1, 0), (0, 2), (2, 1)])
def test_ends(lib, ctx, shape, ends):
    import torch
    d, n = len(shape), int(np.prod(shape))
    rs = np.random.default_rng([n, d, *ends])
    # the ends of successive axes differ; mirrors need three cells
    lo = [ends[a % 2] if shape[a] >= 3 or ends[a % 2] < 2 else 1 for a in range(d)]
    hi = [ends[(a + 1) % 2] if shape[a] >= 3 or ends[(a + 1) % 2] < 2 else 0 for a in range(d)]
    dx = tuple(1.0 / m for m in shape)
    U = wl.prim_to_cons(rs.uniform(1.0, 1.2, n), [rs.uniform(-20.0, 20.0, n) for _ in range(d)],
                        rs.uniform(1e5, 1.1e5, n), rs.uniform(1.4, 1.5, n), rs.uniform(0.0, 1e3, n))
    og, ig = oracle.make_grid(shape, dx, tuple(lo), tuple(hi)), lib.make_grid(shape, dx, lo, hi)
    oo, o, st = oracle.make_opts(), lib.make_opts(), lib.new_stats()
    assert _same_bits(ctx.rhs(_dev(U), ig, o, stats=st).cpu().numpy(), oracle.rhs(U, og, oo)[0])
    V, dt = _dev(U), torch.zeros(1, dtype=torch.float64, device="cuda")
    for _ in range(2):
        ctx.rk3_step(V, ig, o, dt, st)
    W = U
    for _ in range(2):
        W, status = oracle.rk3_step(W, og, oracle.cfl_dt(W, og, oo), oo)
        assert status == 0
    assert _same_bits(V.cpu().numpy(), W)

"""The time step that a 1D step writes is the value of isweno_cfl_dt on U^n,
bit for bit and in both forms, on lines of one launch and longer ones."""
import numpy as np
import pytest

from paper_1707_00592_amd import workloads as wl
from test_gpu_division_ranges import _dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 64, 200, 300, 511, 512, 3000])
@pytest.mark.parametrize("precision", [0, 1])
def test_dt_is_that_of_cfl_dt(lib, n, precision):
    import torch
    ctx = lib.Context(0)
    o = lib.make_opts(precision=precision, cfl=0.37)
    ig = lib.make_grid((n,), (1.0 / n,), 0, 0)
    dt, h = (torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2))
    for seed in range(20):
        # fast cells of one stiffened gas: every product of the speed rounds
        rs = np.random.default_rng(seed)
        U = _dev(wl.prim_to_cons(rs.uniform(0.5, 2, n), [rs.uniform(200, 600, n)],
                                 rs.uniform(1e5, 9e5, n), 1.7, 3e5))
        ctx.cfl_dt(U, ig, o, h)
        ctx.rk3_step(U, ig, o, dt)
        assert float(dt.item()) == float(h.item()), (n, seed)

"""The field-sides counted as linear are those whose tau5 is zero or below
2^-60 epsilon, whichever path evaluated their face: with the cascade off, in
its wave or gathered, and with an epsilon inside or outside the range of the
unscaled divisions."""
import numpy as np
import pytest

from paper_1707_00592_amd import workloads as wl
from test_gpu_division_ranges import _dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-40, 1e-30, 1e-70, 1e40])
def test_counts_do_not_depend_on_the_path(lib, eps):
    p = wl.shock_bubble_2d(96, 64)
    rs = np.random.default_rng(3)
    U = p.U.copy()
    U[0] *= 1 + 1e-18 * rs.random(U.shape[1]) + 1e-17 * rs.integers(0, 40, U.shape[1])
    U[1] += 1e-26 * rs.standard_normal(U.shape[1])  # tau5 below 2^-60 epsilon, but not zero
    m = rs.random(U.shape[1]) < 0.01
    k = int(m.sum())
    U[:, m] = wl.prim_to_cons(rs.uniform(0.5, 1000, k), [rs.uniform(-2000, 2000, k) for _ in range(2)],
                              10 ** rs.uniform(4, 9.4, k), 4.4, 6e8)
    ctx = lib.Context(0)
    ig = lib.make_grid(p.n, p.dx, p.bc_lo, p.bc_hi)
    counts = []
    for mood in (lib.MOOD_OFF, lib.MOOD_ON, lib.MOOD_GATHER):
        ctx.timing_enable(True)
        ctx.rhs(_dev(U), ig, lib.make_opts(mood=mood, eps=eps))
        counts.append(ctx.shortcut_read())
        ctx.timing_enable(False)
    assert counts[0] == counts[1] == counts[2] and min(counts[0][:2]) > 0, counts

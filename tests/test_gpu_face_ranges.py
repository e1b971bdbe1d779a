"""States at the edges of the FP64 faces' common case: the linear form's
tau5 threshold (2^-60 epsilon), and the ranges a tile's cells and a face's
sound speed must lie in for the unscaled divisions, each straddled so that
some tiles, waves and stencils lie on either side.  Bit for bit with the
oracle, with equal MOOD counts, in 1D, 2D and 3D."""
import numpy as np
import pytest

import oracle
from paper_1707_00592_amd import workloads as wl
from test_gpu_division_ranges import FORMS, _check

pytestmark = pytest.mark.gpu

SHAPES = [(300,), (70, 37), (36, 18, 10)]


@pytest.fixture(scope="module")
def ctx(lib):
    return lib.Context(0)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("weights", FORMS)
@pytest.mark.parametrize("eps", [1e-40, 1e12, 1e22, 1e29])
def test_tau5_around_the_linear_threshold(lib, ctx, shape, weights, eps):
    """Amplitudes from 1e-14 to 1 along x: tau5 of every field crosses the
    threshold somewhere for one of the epsilons."""
    rs = np.random.default_rng(len(shape))
    size = np.logspace(-14, 0, shape[0])
    n = int(np.prod(shape))
    s = np.broadcast_to(size, shape[::-1]).ravel()

    def wave():
        return s * rs.uniform(-1, 1, size=n)
    U = wl.prim_to_cons(1000.0 * (1 + 0.1 * wave()), [100.0 * wave() for _ in shape],
                        1e5 * (1 + 0.5 * wave()), 4.4, 6e8)
    _check(lib, ctx, U, shape, weights, eps, "amplitudes 1e-14..1")


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("weights", FORMS)
@pytest.mark.parametrize("edge", ["p", "rho", "c2", "Gamma", "Pi", "u"])
def test_states_across_the_edges_of_the_range(lib, ctx, shape, weights, edge):
    rs = np.random.default_rng(7)
    n = int(np.prod(shape))
    ramp = np.broadcast_to(np.linspace(-1, 1, shape[0]), shape[::-1]).ravel()

    def around(edge_value):  # from 1/100 to 100 times the edge
        return edge_value * 100.0 ** ramp * (1 + 0.01 * rs.uniform(-1, 1, size=n))
    rho, p, G, P = np.ones(n), np.full(n, 1e5), np.full(n, 2.5), np.zeros(n)
    vel = [rs.uniform(-1, 1, size=n) for _ in shape]
    if edge == "p":
        p = around(2.0 ** 40)
    elif edge == "rho":
        rho = around(2.0 ** -20)
    elif edge == "c2":
        p = around(2.0 ** -40)
        vel = [1e-8 * v for v in vel]
    elif edge == "Gamma":
        G = around(2.0 ** 10)
    elif edge == "Pi":
        P = around(2.0 ** 40)
    else:
        p = np.full(n, 2.0 ** 40)
        vel = [around(2.0 ** 24) for _ in shape]
    U = np.ascontiguousarray(np.stack(
        [rho, *[rho * v for v in vel], G * p + P + 0.5 * rho * sum(v * v for v in vel), G, P]))
    _check(lib, ctx, U, shape, weights, 1e-40, f"edge of {edge}")

"""dJ/dA of one reverse step against its closed form in FP64 on the same stored inputs.

A enters a step through the perturbation A |grad phi| [w_i (c_i.n)^2 - B_i] alone, so
dJ/dA is a sum over the nodes of |grad phi| sum_i L'_i [w_i (c_i.n)^2 - B_i], L' the
colour-blind cotangents of the post-collision populations.  The terms of the nodes
alternate in sign, and the sum keeps the absolute rounding of each: with cotangents,
fields and colour fractions as the library stores them (FP32), it has to be an FP64
sum of FP64 terms.

Tolerance: about 40 FP64 operations per node and at most 100 additions on the way to
the total, 140 * 2^-53 = 1.6e-14 of the sum of the terms' magnitudes; 1e-13 is taken.
FP32 terms are about 1e-9 off on these lattices.
"""
import numpy as np
import pytest

from harness import Q, say
from test_gpu_adjoint import _gpu_adjoint, _jet, _periodic, _state, torch  # noqa: F401

pytestmark = pytest.mark.gpu

# the last: ten tiles a plane, so that blocks of its launch lie beyond the last plane
SHAPES = [(65, 7, 9), (129, 9, 8), (20, 37, 7)]


@pytest.mark.parametrize("bc", ["periodic", "jet"])
@pytest.mark.parametrize("shape", SHAPES)
def test_dA_in_fp64(torch, orc, shape, bc):  # noqa: F811
    nx, ny, nz = shape
    prob = _jet(nx, ny, nz, D=1.5) if bc == "jet" else _periodic(nx, ny, nz)
    st32, st = _state(orc, prob, seed=nx)
    rng = np.random.default_rng(nx + 7)
    w32 = rng.standard_normal(st32.shape).astype(np.float32)
    grid = w32.reshape(2, Q, nz, ny, nx)
    if bc == "jet":  # away from the walls, the inlet and the outlet: streaming is a shift there
        keep = np.zeros((nz, ny, nx), bool)
        keep[2:-3, 2:-2, 2:-2] = True
        grid *= keep
    dA = _gpu_adjoint(torch, prob, st32, 5, w32)[1]

    c, w = orc.lattice()
    c, w = np.asarray(c), np.asarray(w, np.float64)
    rr, rho = st[:Q].sum(0), st.sum(0)
    a, b = rr * prob.rho_b0, (rho - rr) * prob.rho_r0
    phi = ((a - b) / (a + b)).astype(np.float32).astype(np.float64).reshape(nz, ny, nx)
    xr = (rr / rho).astype(np.float32).astype(np.float64).reshape(nz, ny, nx)

    def ahead(f, i):  # f at x + c_i
        return np.roll(f, (-c[i][2], -c[i][1], -c[i][0]), (0, 1, 2))
    g = [sum(3.0 * w[i] * c[i][d] * ahead(phi, i) for i in range(1, Q)) for d in range(3)]
    gn = np.sqrt(sum(q * q for q in g))
    total, scale = 0.0, 0.0
    for i in range(Q):
        lr, lb = (ahead(grid[k, i].astype(np.float64), i) for k in (0, 1))
        cn = sum(int(c[i][d]) * g[d] for d in range(3)) / gn
        t = gn * (lb + xr * (lr - lb)) * (w[i] * cn * cn - (-10.0 / 27.0 if i == 0 else w[i]))
        total += t.sum()
        scale += np.abs(t).sum()
    say(f"dJ/dA {bc} {shape}: {dA:.12e} against {total:.12e}, off by {abs(dA - total) / scale:.1e} of the terms")
    assert abs(dA - total) <= 1e-13 * scale

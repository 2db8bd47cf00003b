"""The reverse step at the edges of its tiles: row lengths around the 64-node
segments and the 128-node tiles (a row that ends inside a wavefront, one node into
the next tile, several tiles), with the walls, the wrapped columns, the inlet and the
planes under the outlet in wavefronts of their own.

<w, J v> = <J^T w, v> against the FP64 oracle's complex step, v random and v on
the columns next to the walls and segment ends.  The node arithmetic is FP32, so the
products agree to 2e-6 of the sum of their terms' magnitudes.
"""
import numpy as np
import pytest

from harness import say
from test_gpu_adjoint import _cs_step, _gpu_adjoint, _inlet_profile, _jet, _periodic, _state, torch  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [(63, 3, 4), (64, 6, 4), (65, 4, 3), (127, 3, 4), (128, 5, 5), (129, 4, 3), (193, 3, 3)]


@pytest.mark.parametrize("bc", ["periodic", "jet"])
@pytest.mark.parametrize("shape", SHAPES)
def test_adjoint_rows(torch, orc, orc_cs, shape, bc):  # noqa: F811
    nx, ny, nz = shape
    prob = _jet(nx, ny, nz, D=1.5) if bc == "jet" else _periodic(nx, ny, nz)
    st32, st64 = _state(orc, prob, seed=nx)
    rng = np.random.default_rng(nx + 1)
    w32 = rng.standard_normal(st32.shape).astype(np.float32)
    inlet = _inlet_profile(prob, 2) if bc == "jet" else None
    lam, dA, du = _gpu_adjoint(torch, prob, st32, 9, w32, inlet)
    w64 = w32.astype(np.float64)
    x = np.tile(np.arange(nx), ny * nz)
    ends = (x == 0) | (x == nx - 1) | (x % 64 == 0) | (x % 64 == 63)
    for kind in ("random", "ends"):
        v = rng.standard_normal(st64.shape)
        if kind == "ends":
            v[:, ~ends] = 0.0
        lhs = (w64 * _cs_step(orc_cs, prob, st64, 9, v=v, inlet=inlet)).sum()
        rhs, scale = (lam * v).sum(), np.abs(lam * v).sum()
        say(f"adjoint rows {bc} {shape} {kind}: err/sum|lam v| {abs(rhs - lhs) / scale:.2e}")
        assert abs(rhs - lhs) <= 2e-6 * scale
    d = _cs_step(orc_cs, prob, st64, 9, dA=1.0, inlet=inlet)
    assert abs(dA - (w64 * d).sum()) <= 2e-6 * np.abs(w64 * d).sum()


def test_adjoint_beyond_the_caches(torch, orc):  # noqa: F811
    """Cotangents that do not fit the memory-side cache are stored past it: a periodic
    lattice of 40 equal slabs (1.3 M nodes, 283 MB of cotangents) against one slab.
    The nodes' arithmetic is the same, so they agree to FP32 rounding."""
    small, slabs = _periodic(64, 64, 8), 40
    st32, _ = _state(orc, small, seed=3)
    w32 = np.random.default_rng(4).standard_normal(st32.shape).astype(np.float32)
    ref, dA, _ = _gpu_adjoint(torch, small, st32, 5, w32)
    big = _periodic(64, 64, 8 * slabs)
    lam, dA_big, _ = _gpu_adjoint(torch, big, np.tile(st32, slabs), 5, np.tile(w32, slabs))
    err = np.abs(lam.reshape(len(ref), slabs, -1) - ref[:, None, :]).max() / np.abs(ref).max()
    say(f"adjoint of {slabs} equal slabs: max difference {err:.2e}, dJ/dA {dA_big:.9e} against {slabs * dA:.9e}")
    assert err <= 1e-6
    assert abs(dA_big - slabs * dA) <= 1e-6 * abs(slabs * dA)

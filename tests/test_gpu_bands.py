"""Launches whose blocks stand in one row, in bands for the eight XCDs: nine tiles a plane
or more and no multiple of eight, with blocks beyond the last plane.  The step in every
storage and the reverse step against the FP64 oracle, on both boundary kinds; tiles a
plane, planes (density, fused, adjoint; 64x8, 64x4 of the referenced 16-bit forms):

  20x75x5   19 narrow tiles, 10 of the referenced forms' density tiles
  100x37x5  10 wide density tiles, 19 wide fused tiles
  129x30x6  24 narrow (no bands), 12 of the referenced forms' density tiles

The row lengths on both sides of a tile's end in the 16-bit storages that the row tests
leave out, and a jet's reverse step whose cotangents do not fit the memory-side cache.
"""
import numpy as np
import pytest

from harness import Q, hist_from, random_state, say, state_to_f32
from test_gpu_adjoint import _cs_step, _gpu_adjoint, _inlet_profile, _jet, _periodic, _state, torch  # noqa: F401
from test_gpu_rows import _problem

pytestmark = pytest.mark.gpu

BANDS = [(20, 75, 5), (100, 37, 5), (129, 30, 6)]
EDGES = [(63, 3, 4), (65, 4, 3), (127, 3, 4), (128, 4, 3), (129, 4, 3), (193, 3, 3)]
CASES = [(s, k) for s in BANDS for k in ("fp32", "bf16", "fp16", "bf16eq", "fp16eq")]
CASES += [(s, k) for s in EDGES for k in ("bf16", "fp16", "bf16eq")]


@pytest.mark.parametrize("bc", ["periodic", "jet"])
@pytest.mark.parametrize("shape,storage", CASES)
def test_step_against_oracle(orc, shape, storage, bc):
    import torch as t

    from paper_1804_08923_amd.lbm import LBM
    prob = _problem(shape, bc, storage)
    p, fr, fb, _ = random_state(orc, prob, seed=sum(shape))
    sim = LBM(prob)
    sim.set_state(t.from_numpy(state_to_f32(fr, fb)[0]).cuda(), t=3)
    held = sim.get_state().cpu().numpy().astype(np.float64)
    fr, fb = held[:Q].copy(), held[Q:].copy()
    orc.step(p, prob.A, fr, fb, hist_from(p, fr, fb), 3, 2)
    sim.step(2)
    got = sim.get_state().cpu().numpy().astype(np.float64)
    sim.close()
    scale = np.abs(fr + fb).max()
    err = max(np.abs(got[:Q] - fr).max(), np.abs(got[Q:] - fb).max()) / scale
    # FP32: 1e-6 a step; 16 bits: a spacing (2^-8, 2^-11 relative) of a stored deviation
    # per step
    tol = 2e-6
    if storage != "fp32":
        w = np.asarray(orc.lattice()[1], np.float64)
        dev = np.abs(fr + fb - w[:, None] * prob.rho_b0).max()
        tol += 2 * (2.0 ** -8 if storage[:4] == "bf16" else 2.0 ** -11) * dev / scale
    say(f"  {shape} {storage} {bc}: max pop err {err:.2e} (tolerance {tol:.2e})")
    assert err < tol


@pytest.mark.parametrize("bc", ["periodic", "jet"])
@pytest.mark.parametrize("shape", BANDS)
def test_reverse_step_against_oracle(torch, orc, orc_cs, shape, bc):  # noqa: F811
    """<w, J v> = <J^T w, v> as in the reverse step's row tests: 2e-6 of the terms."""
    nx, ny, nz = shape
    prob = _jet(nx, ny, nz, D=4.0) if bc == "jet" else _periodic(nx, ny, nz)
    st32, st64 = _state(orc, prob, seed=nx)
    rng = np.random.default_rng(nx + 1)
    w32 = rng.standard_normal(st32.shape).astype(np.float32)
    inlet = _inlet_profile(prob, 2) if bc == "jet" else None
    lam, dA, _ = _gpu_adjoint(torch, prob, st32, 9, w32, inlet)
    w64 = w32.astype(np.float64)
    z = np.repeat(np.arange(nz), nx * ny)
    for kind, sel in (("all", z >= 0), ("last planes", z >= nz - 2)):
        v = rng.standard_normal(st64.shape) * sel
        lhs = (w64 * _cs_step(orc_cs, prob, st64, 9, v=v, inlet=inlet)).sum()
        rhs, scale = (lam * v).sum(), np.abs(lam * v).sum()
        say(f"  {shape} {bc} {kind}: err/sum|lam v| {abs(rhs - lhs) / scale:.2e}")
        assert abs(rhs - lhs) <= 2e-6 * scale
    d = _cs_step(orc_cs, prob, st64, 9, dA=1.0, inlet=inlet)
    assert abs(dA - (w64 * d).sum()) <= 2e-6 * np.abs(w64 * d).sum()


def test_jet_reverse_step_beyond_the_caches(torch, orc):  # noqa: F811
    """1.3 M nodes, 283 MB of cotangents, stored past the caches.  What a reverse step
    writes at a node depends on the planes up to three away: the lowest planes equal
    those of a short jet cut from the bottom, the highest those of one cut from the top.
    The arithmetic is the same; the bound is FP32 rounding."""
    nx, ny, cut, mid = 64, 64, 16, 296
    P = nx * ny
    a, _ = _state(orc, _jet(nx, ny, cut, D=8.0), seed=5)
    b, _ = _state(orc, _jet(nx, ny, cut, D=8.0), seed=6)
    rng = np.random.default_rng(7)
    wa, wb = (rng.standard_normal(a.shape).astype(np.float32) for _ in range(2))
    big = _jet(nx, ny, 2 * cut + mid, D=8.0, noise=0.0)
    short = _jet(nx, ny, cut, D=8.0, noise=0.0)

    def stack(low, high):  # low, its top plane repeated, high
        return np.concatenate([low, np.tile(low[:, -P:], mid), high], axis=1)
    lam, _, du = _gpu_adjoint(torch, big, stack(a, b), 5, stack(wa, wb))
    low, _, du_low = _gpu_adjoint(torch, short, a, 5, wa)
    high, _, _ = _gpu_adjoint(torch, short, b, 5, wb)
    n = (cut - 4) * P
    scale = np.abs(low).max()
    errs = (np.abs(lam[:, :n] - low[:, :n]).max() / scale, np.abs(lam[:, -n:] - high[:, -n:]).max() / scale,
            np.abs(du - du_low).max() / np.abs(du_low).max())
    say("  lowest planes off by {:.1e}, highest by {:.1e}, dJ/du by {:.1e}".format(*errs))
    assert max(errs) <= 1e-6

"""Rows that leave many lanes of a tile idle: the state-reading kernels (macroscopic
fields, get_state, diagnostics) and the D3Q19 step change to blocks of consecutive nodes
there, at row lengths of their own.  On both sides of each of those lengths, on both
boundary kinds: two steps against the FP64 oracle, the macroscopic fields against the
FP64 sums of the state that get_state returns, the diagnostics against the CPU reference
on the GPU's own phi.  Lattices of one and two rows are among the periodic ones.

And what the choice is for: a report of a narrow lattice costs no more than a few times
that of a wide one with as many nodes.
"""
import numpy as np
import pytest

from harness import hist_from, say
from oracle import Oracle
from oracle import make_params as or_params
from oracle.diagnostics import jet_diagnostics
from paper_1804_08923_amd.workloads import Problem

pytestmark = pytest.mark.gpu

SHAPES = [(1, 7, 9), (2, 1, 6), (5, 2, 3), (3, 5, 4), (15, 4, 5), (16, 6, 3), (23, 3, 4), (24, 4, 3), (31, 5, 3),
          (32, 3, 4), (35, 4, 3), (36, 3, 5), (43, 3, 4), (44, 5, 3), (71, 3, 4), (72, 4, 3), (87, 3, 4), (88, 3, 3)]


def _problem(shape, bc, storage, lattice):
    nx, ny, nz = shape
    jet = dict(inlet_cx=(nx - 1) / 2.0, inlet_cy=(ny - 1) / 2.0, inlet_D=0.9, inlet_u=0.04, noise_amp=0.02,
               noise_seed=11) if bc == "jet" else {}
    return Problem(name="narrow", nx=nx, ny=ny, nz=nz, bc=bc, rho_r0=1.0, rho_b0=0.5, nu_r=0.02, nu_b=0.05, A=2e-3,
                   g=(0.0, 0.0, 3e-4) if bc == "jet" else (1e-4, -2e-4, 3e-4), init="jet", storage=storage,
                   lattice=lattice, alpha_b=8 / 27 if lattice == 27 else 1 / 3, **jet)


@pytest.mark.parametrize("kind", ["fp32", "bf16", "fp16", "bf16eq", "fp16eq", "d3q19"])
@pytest.mark.parametrize("shape,bc", [(s, b) for s in SHAPES for b in ("periodic", "jet")
                                      if b == "periodic" or min(s) >= 3])  # the jet needs three nodes an axis
def test_narrow_rows(orc, shape, kind, bc):
    import torch

    from paper_1804_08923_amd.lbm import LBM
    from synth import random_state_fields
    q19 = kind == "d3q19"
    Q = 19 if q19 else 27
    ref = Oracle("q19") if q19 else orc
    prob = _problem(shape, bc, "fp32" if q19 else kind, Q)
    p = or_params(prob)
    fr, fb, _ = ref.init_fields(p, *random_state_fields(prob, sum(shape)))
    sim = LBM(prob)
    sim.set_state(torch.from_numpy(np.concatenate([fr, fb]).astype(np.float32)).cuda(), t=3)
    held = sim.get_state().cpu().numpy().astype(np.float64)
    fr, fb = held[:Q].copy(), held[Q:].copy()
    P = prob.nx * prob.ny
    hist = np.concatenate([fr[:, -P:], fb[:, -P:]]) if q19 else hist_from(p, fr, fb)
    ref.step(p, prob.A, fr, fb, hist, 3, 2)
    sim.step(2)
    got = sim.get_state().cpu().numpy().astype(np.float64)
    m = {a: v.cpu().numpy().astype(np.float64) for a, v in sim.macroscopic().items()}
    stats, vol = sim.jet_diagnostics()
    sim.close()
    scale = np.abs(fr + fb).max()
    # FP32: 1e-6 a step; 16 bits: half a spacing (2^-9, 2^-12 relative) of a stored
    # deviation per step
    tol = 2e-6
    w = np.asarray(ref.lattice()[1], np.float64)
    if kind[:4] in ("bf16", "fp16"):
        tol += 2 * (2.0 ** -8 if kind[:4] == "bf16" else 2.0 ** -11) * np.abs(fr + fb - w[:, None] * prob.rho_b0).max() / scale
    err = max(np.abs(got[:Q] - fr).max(), np.abs(got[Q:] - fb).max()) / scale
    # the fields are FP32 values of FP64 sums; get_state rounds every population (2^-24)
    rr, rb = got[:Q].sum(0), got[Q:].sum(0)
    off = max(np.abs(m["rho_r"] - rr).max(), np.abs(m["rho_b"] - rb).max()) / (rr + rb).max()
    say(f"  {shape} {kind} {bc}: max pop err {err:.2e} (tolerance {tol:.2e}), densities {off:.2e}")
    assert err < tol
    assert off < 4 * 2.0 ** -24
    want, want_vol = jet_diagnostics(m["phi"].astype(np.float32), *shape)
    assert stats == want and np.array_equal(vol, want_vol)


def _ms(torch, call, n=20):
    for _ in range(3):
        call()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(n):
        call()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b) / n


def test_narrow_lattices_cost_a_few_times_wide_ones():
    """10^6 nodes; measured ratios 3.7, 2.8 and 1.4 (18, 17 and 5 by tiles alone), and 0.9
    for a state whose rows are not padded to whole lines (1.6 with rows of 64)."""
    import torch

    from paper_1804_08923_amd.lbm import LBM

    def cost(nx, nz, lattice, what):
        sim = LBM(_problem((nx, 128, nz), "periodic", "fp32", lattice))
        sim.step(2)
        return _ms(torch, dict(step=lambda: sim.step(1), fields=sim.macroscopic, state=sim.get_state)[what])
    for lattice, what, nx, nz, most in ((27, "fields", 3, 2730, 8.0), (19, "fields", 3, 2730, 8.0),
                                        (19, "step", 8, 1024, 3.0), (19, "state", 40, 204, 1.25)):
        ratio = cost(nx, nz, lattice, what) / cost(128, 64, lattice, what)
        say(f"  D3Q{lattice} {what}: {nx}x128x{nz} costs {ratio:.1f} times 128x128x64")
        assert ratio < most

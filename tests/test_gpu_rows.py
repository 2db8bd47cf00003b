"""The row layout of a running state against the FP64 oracle: row lengths around
the 64-node segments and 128-node tiles of the step kernels (a tile whose right
rim lies inside it, one node into the next tile, several tiles), strides that are
longer than the row and strides that cannot be aligned, on both boundary kinds
(lattices of one and two rows: test_gpu_narrow_rows.py).

Three steps from a random state: the first reads the state as it was set, the
others read rows.  D3Q19 shares the layout and is held to its own oracle.
"""
import numpy as np
import pytest

from harness import Q, hist_from, random_state, say, state_to_f32
from paper_1804_08923_amd.workloads import Problem

pytestmark = pytest.mark.gpu

SHAPES = [(62, 5, 4), (63, 3, 3), (64, 8, 8), (65, 4, 3), (127, 3, 4), (128, 5, 3), (129, 4, 3), (193, 3, 3)]


def _problem(shape, bc, storage, lattice=27):
    nx, ny, nz = shape
    jet = dict(inlet_cx=(nx - 1) / 2.0, inlet_cy=(ny - 1) / 2.0, inlet_D=1.5, inlet_u=0.04, noise_amp=0.02,
               noise_seed=11) if bc == "jet" else {}
    return Problem(name="rows", nx=nx, ny=ny, nz=nz, bc=bc, rho_r0=1.0, rho_b0=0.5, nu_r=0.02, nu_b=0.05, A=2e-3,
                   g=(0.0, 0.0, 3e-4) if bc == "jet" else (1e-4, -2e-4, 3e-4), init="jet", storage=storage, lattice=lattice,
                   alpha_b=8 / 27 if lattice == 27 else 1 / 3, **jet)


@pytest.mark.parametrize("bc", ["periodic", "jet"])
@pytest.mark.parametrize("storage", ["fp32", "fp16eq"])
@pytest.mark.parametrize("shape", SHAPES)
def test_rows_against_oracle(orc, shape, storage, bc):
    import torch

    from paper_1804_08923_amd.lbm import LBM
    prob = _problem(shape, bc, storage)
    p, fr, fb, _ = random_state(orc, prob, seed=sum(shape))
    sim = LBM(prob)
    sim.set_state(torch.from_numpy(state_to_f32(fr, fb)[0]).cuda(), t=3)
    # the oracle starts from what the library holds (the storage rounds it)
    held = sim.get_state().cpu().numpy().astype(np.float64)
    fr, fb = held[:Q].copy(), held[Q:].copy()
    orc.step(p, prob.A, fr, fb, hist_from(p, fr, fb), 3, 3)
    sim.step(3)
    got = sim.get_state().cpu().numpy().astype(np.float64)
    sim.close()
    scale = np.abs(fr + fb).max()
    err = max(np.abs(got[:Q] - fr).max(), np.abs(got[Q:] - fb).max()) / scale
    # FP32: 1e-6 a step, the bar of the other parity tests.  FP16 remainders: half
    # a spacing (2^-11 relative) of a remainder per step; the remainders are below
    # the deviations of the moving directions
    tol = 3e-6
    if storage == "fp16eq":
        w = np.asarray(orc.lattice()[1], np.float64)
        tol += 3 * 2.0 ** -11 * np.abs(fr + fb - w[:, None] * prob.rho_b0)[1:].max() / scale
    say(f"  {shape} {storage} {bc}: max pop err {err:.2e} (tolerance {tol:.2e})")
    assert err < tol


@pytest.mark.parametrize("bc", ["periodic", "jet"])
@pytest.mark.parametrize("shape", SHAPES)
def test_q19_rows_against_oracle(shape, bc):
    import torch

    from oracle import Oracle
    from oracle import make_params as or_params
    from paper_1804_08923_amd.lbm import LBM
    from synth import random_state_fields
    orc = Oracle("q19")
    prob = _problem(shape, bc, "fp32", lattice=19)
    p = or_params(prob)
    fr, fb, _ = orc.init_fields(p, *random_state_fields(prob, sum(shape)))
    sim = LBM(prob)
    sim.set_state(torch.from_numpy(np.concatenate([fr, fb]).astype(np.float32)).cuda(), t=3)
    held = sim.get_state().cpu().numpy().astype(np.float64)
    fr, fb = held[:19].copy(), held[19:].copy()
    P = prob.nx * prob.ny
    orc.step(p, prob.A, fr, fb, np.concatenate([fr[:, -P:], fb[:, -P:]]), 3, 3)
    sim.step(3)
    got = sim.get_state().cpu().numpy().astype(np.float64)
    sim.close()
    err = max(np.abs(got[:19] - fr).max(), np.abs(got[19:] - fb).max()) / np.abs(fr + fb).max()
    say(f"  D3Q19 {shape} {bc}: max pop err {err:.2e}")
    assert err < 3e-6  # 1e-6 a step, as above

"""A lattice of one node along x with 2^26 rows: its 64x4 and 128x2 tiles are more than
one row of blocks can hold (2^32 lanes), so the launches keep a row of blocks per plane.

The lattice repeats a small periodic one along y and z.  Every node's arithmetic is the
same on the same inputs, so its fields equal the small lattice's bit for bit.
"""
import numpy as np
import pytest

from harness import say
from paper_1804_08923_amd.workloads import Problem

pytestmark = pytest.mark.gpu

NY, NZ, KY, KZ = 92, 72, 89, 114


def _run(torch, ny, nz, phi):
    from paper_1804_08923_amd.lbm import LBM
    prob = Problem(name="thin", nx=1, ny=ny, nz=nz, rho_r0=1.0, rho_b0=0.5, nu_r=0.02, nu_b=0.05, A=2e-3,
                   g=(0.0, 0.0, 1e-5), init="fields", storage="fp16")
    sim = LBM(prob, rho_r=0.5 * (1 + phi.reshape(-1)), rho_b=0.25 * (1 - phi.reshape(-1)))
    sim.step(2)
    out = sim.macroscopic()
    stats, _ = sim.jet_diagnostics()
    sim.close()
    return out, stats


def test_more_lanes_than_one_row_of_blocks():
    import torch
    rng = np.random.default_rng(26)
    phi = torch.from_numpy(np.tanh(rng.standard_normal((NZ, NY))).astype(np.float32)).cuda()
    small, few = _run(torch, NY, NZ, phi)
    big, many = _run(torch, NY * KY, NZ * KZ, phi.repeat(KZ, KY))
    say(f"jet nodes {few['jet_nodes']} in the small lattice, {many['jet_nodes']} in {KY * KZ} of them")
    assert many["jet_nodes"] == KY * KZ * few["jet_nodes"]
    for name in ("rho_r", "rho_b", "phi", "u"):
        a = small[name].reshape(NZ, NY, -1)
        b = big[name].reshape(KZ, NZ, KY, NY, -1)
        assert bool((b == a[None, :, None]).all()), name

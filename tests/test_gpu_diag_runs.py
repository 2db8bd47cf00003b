"""The union-find of the jet diagnostics where its runs along x begin and end: row
lengths around the 64-node segments, on both lattices, and lattices with fewer
planes than a counting thread takes and with a remainder.  Site-percolation fields (every node drawn by
itself) make runs of every length and components that join through all three
axes.  Whole numbers, compared exactly with the CPU reference on the GPU's own phi.
"""
import numpy as np
import pytest

from oracle.diagnostics import jet_diagnostics
from paper_1804_08923_amd.workloads import Problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lattice", [27, 19])
@pytest.mark.parametrize("share", [0.2, 0.32, 0.9])
@pytest.mark.parametrize("shape", [(63, 5, 7), (64, 4, 16), (65, 6, 17), (129, 3, 33), (200, 7, 5), (7, 40, 18)])
def test_percolation_components(shape, share, lattice):
    import torch

    from paper_1804_08923_amd.lbm import LBM
    nx, ny, nz = shape
    rng = np.random.default_rng(sum(shape) + int(100 * share) + lattice)
    phi = np.where(rng.random(nx * ny * nz) < share, 0.8, -0.8)
    prob = Problem(name="perc", nx=nx, ny=ny, nz=nz, rho_r0=1.0, rho_b0=0.5, init="fields", lattice=lattice,
                   alpha_b=8 / 27 if lattice == 27 else 1 / 3)
    sim = LBM(prob, rho_r=torch.from_numpy((0.5 * (1 + phi)).astype(np.float32)),
              rho_b=torch.from_numpy((0.25 * (1 - phi)).astype(np.float32)))
    for _ in range(2):  # the state as it was set, then rows
        stats, vol = sim.jet_diagnostics()
        ref, rvol = jet_diagnostics(sim.macroscopic()["phi"].cpu().numpy(), nx, ny, nz)
        assert stats == ref
        assert np.array_equal(vol, rvol)
        sim.step(1)
    sim.close()

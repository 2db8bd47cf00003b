"""The launch grids of the tiled kernels and the order of their blocks, on the host.

Every lattice that the parameters admit (2^29 padded nodes, 65535 a dimension) has to
give a grid that can be launched: fewer than 2^32 lanes along x, at most 65535 blocks
along y.  Every tile of every plane has to be taken by exactly one block.
"""
import os
import subprocess

import pytest

from paper_1804_08923_amd.build import CSRC, HIPCC_FLAGS, ROOT

HERE = os.path.dirname(os.path.abspath(__file__))
PACKED = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
TILES = [(128, 2), (128, 4), (64, 4), (64, 8)]


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("native") / "tile_grid_check")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", *HIPCC_FLAGS[:1], "-O1", "-std=c++17",
                    *PACKED, "-w", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", exe,
                    os.path.join(HERE, "native", "tile_grid_check.cpp")], check=True)

    def run(lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", text=True, capture_output=True, check=True).stdout
        return [[int(v) for v in row.split()] for row in out.splitlines()]
    return run


def _thin():
    """The longest lattices for each small nx, ny on and next to multiples of eight tiles."""
    for nx in (1, 2, 3, 5, 12, 13, 63, 64, 65, 129):
        for ny in (64, 1001, 2340, 4679, 4680, 8188, 16375, 23001, 32768, 65500, 65535):
            nz = min(65535, 2 ** 29 // ((nx + 2) * (ny + 2)) - 2)
            if nz >= 1:
                yield nx, ny, nz
    yield 12, 4679, 8190
    yield 65535, 1363, 4


def test_every_grid_can_be_launched(check):
    shapes = list(_thin())
    got = check([f"limits {nx} {ny} {nz}" for nx, ny, nz in shapes])
    assert len(got) == len(TILES) * len(shapes)
    for k, (lanes, gx, gy, gz) in enumerate(got):
        what = shapes[k // len(TILES)], TILES[k % len(TILES)], (gx, gy, gz)
        assert lanes < 2 ** 32 and 1 <= gy <= 65535 and gz == 1, what


def test_every_tile_once(check):
    shapes = [(nx, ny, nz) for nx in (1, 64, 65, 129, 300) for ny in (1, 7, 16, 33, 36, 37, 75, 130)
              for nz in (1, 2, 5, 7, 8, 9, 17)]
    shapes.append((1, 8188, 8208))  # past the limit of one row with 64x4 tiles
    got = check([f"visit {nx} {ny} {nz}" for nx, ny, nz in shapes])
    assert len(got) == len(TILES) * len(shapes)
    assert not any(w for (w,) in got), [(shapes[k // len(TILES)], TILES[k % len(TILES)])
                                        for k, (w,) in enumerate(got) if w]


def test_audit_of_a_thin_lattice_is_small():
    """One slot of five doubles per block of 256 nodes, not per two rows of a tile."""
    from paper_1804_08923_amd.lbm import lbm_query_sizes, make_params
    from paper_1804_08923_amd.workloads import Problem
    for lattice in (27, 19):
        prob = Problem(name="thin", nx=1, ny=4096, nz=4096, rho_r0=1.0, rho_b0=0.5, nu_r=0.02, nu_b=0.05, init="jet",
                       lattice=lattice, alpha_b=8 / 27 if lattice == 27 else 1 / 3)
        s = lbm_query_sizes(make_params(prob))
        assert s.audit_bytes <= 40 * (s.n_nodes // 256 + 1)

"""Parity of the HIP path (through the C ABI) with the FP64 oracle.

Element-by-element comparisons on seeded inputs at sizes the oracle finishes
in seconds (several 256-node blocks plus a ragged tail).  Tolerances: the
target rel L-inf <= 1e-5 on density and velocity after 200 steps of
the 32^3 droplet; single steps are compared population by population.
"""
import numpy as np
import pytest

from harness import (Q, gpu_fields, oracle_fields, oracle_init, random_state, rel_linf, say,
                     state_to_f32)
from oracle import make_params as or_params
from paper_1804_08923_amd.workloads import Problem, droplet_cm, droplet_small

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a visible ROCm device"
    return t


def _sim(prob, **kw):
    from paper_1804_08923_amd.lbm import LBM
    return LBM(prob, **kw)


def _gpu_state(sim):
    st = sim.get_state().cpu().numpy().astype(np.float64)
    return st[:Q], st[Q:]


def _periodic_random_problem(nx, ny, nz, **kw):
    base = dict(name="rand", nx=nx, ny=ny, nz=nz, bc="periodic", rho_r0=1.0, rho_b0=0.5,
                nu_r=0.02, nu_b=0.05, A=2e-3, g=(1e-4, -2e-4, 3e-4), init="jet")
    base.update(kw)
    return Problem(**base)


@pytest.mark.parametrize("shape", [(16, 12, 10), (13, 7, 5), (32, 32, 1), (130, 16, 5)])
def test_single_step_random_state(torch, orc, shape):
    """One step from a random physical state (tau != 1, gamma = 2, eta != 1, g != 0):
    every population of both colours against the oracle.  130x16x5 has three
    64-node tiles per row (the last ragged) and 12 tiles per plane, so that the
    blocks stand in one row in bands for the XCDs."""
    prob = _periodic_random_problem(*shape)
    say(f"single step {shape}")
    p, fr, fb, h = random_state(orc, prob, seed=sum(shape))
    st, fr64, fb64 = state_to_f32(fr, fb)
    sim = _sim(prob)
    sim.set_state(torch.from_numpy(st).cuda(), t=0)
    # the state is taken over up to the FP32 rounding of d = f - w rho_b0: each
    # node keeps its minority colour exactly, the other is recovered as
    # (d + w rho_b0) - f^k (a few ulps of max |f|)
    g0r, g0b = _gpu_state(sim)
    fmax = np.abs(fr64 + fb64).max()
    blue = fr64.sum(0) > fb64.sum(0)
    ek = np.where(blue, g0b - fb64, g0r - fr64)
    eo = np.where(blue, g0r - fr64, g0b - fb64)
    assert np.abs(ek).max() == 0.0
    assert np.abs(eo).max() <= 4 * 2.0 ** -23 * fmax
    sim.step(1)
    gr, gb = _gpu_state(sim)
    orc.step(p, prob.A, fr64, fb64, np.zeros((2 * Q, p.nx * p.ny)), 0, 1)
    scale = np.abs(fr64 + fb64).max()
    err_r = np.abs(gr - fr64).max() / scale
    err_b = np.abs(gb - fb64).max() / scale
    say(f"  pop err red {err_r:.2e} blue {err_b:.2e}")
    assert err_r < 2e-6 and err_b < 2e-6
    fo = oracle_fields(orc, p, fr64, fb64)
    fg = gpu_fields(sim)
    errs = {k: rel_linf(fg[k], fo[k]) for k in ("rho", "u", "phi")}
    say(f"  rel Linf {errs}")
    # the FP32 input state is converted to (d, f^r) once (one rounding of d)
    for k, e in errs.items():
        assert e < 1e-5, k


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 6, 4), (5, 1, 3), (3, 4, 1), (129, 2, 2)])
def test_degenerate_periodic_lattices(torch, orc, shape):
    """Lattices one node thick along some axis (a node is then its own
    neighbour across the periodic wrap, and both ghost faces of that axis copy
    the same node), and a row one node wider than a 128-node tile: 10 steps
    from a random state against the oracle, populations of both colours."""
    prob = _periodic_random_problem(*shape)
    say(f"degenerate lattice {shape}")
    p, fr, fb, h = random_state(orc, prob, seed=3 + sum(shape))
    st, fr64, fb64 = state_to_f32(fr, fb)
    sim = _sim(prob)
    sim.set_state(torch.from_numpy(st).cuda(), t=0)
    sim.step(10)
    gr, gb = _gpu_state(sim)
    sim.close()
    orc.step(p, prob.A, fr64, fb64, np.zeros((2 * Q, p.nx * p.ny)), 0, 10)
    scale = np.abs(fr64 + fb64).max()
    err = max(np.abs(gr - fr64).max(), np.abs(gb - fb64).max()) / scale
    say(f"  max pop err {err:.2e}")
    assert err < 1e-5


def test_zero_steps_is_a_no_op(torch, orc):
    prob = _periodic_random_problem(8, 6, 4)
    _, fr, fb, _ = random_state(orc, prob, seed=9)
    st, _, _ = state_to_f32(fr, fb)
    sim = _sim(prob)
    sim.set_state(torch.from_numpy(st).cuda(), t=5)
    before = sim.get_state().cpu().numpy()
    sim.step(0)
    assert sim.time == 5
    assert np.array_equal(sim.get_state().cpu().numpy(), before)
    sim.close()


def _internal_state(sim, prob):
    """The GPU's stored state right after set_state (general form at each node of the
    padded lattice): d_i = f_i - w_i rho_b0 and the populations f^k_i of the node's
    minority colour in FP32 (which colour: lowest bit of the first float of the
    node's recolouring record in the field buffer), converted exactly to (fr, fb)
    in FP64 for the oracle."""
    from harness import Q as _Q
    t = torch_mod()
    shape = (prob.nz + 2, prob.ny + 2, prob.nx + 2)
    NP = shape[0] * shape[1] * shape[2]
    raw = sim.pop_a.view(t.float32)[: 2 * _Q * NP].reshape(2 * _Q, *shape)
    # interior of the padded lattice, node order
    raw = raw[:, 1:-1, 1:-1, 1:-1].reshape(2 * _Q, -1).cpu().numpy().astype(np.float64)
    rx = sim.fields[: 4 * NP].reshape(NP, 4)[:, 0].contiguous().view(t.int32).reshape(shape)
    blue = (rx[1:-1, 1:-1, 1:-1].reshape(-1).cpu().numpy() & 1).astype(bool)
    from oracle import Oracle
    _, w = Oracle("f64").lattice()
    d, fk = raw[:_Q], raw[_Q:]
    fo = d + w[:, None] * prob.rho_b0 - fk
    return np.where(blue, fo, fk), np.where(blue, fk, fo)


def torch_mod():
    import torch as t
    return t


@pytest.mark.parametrize("gz", [0.0, 3e-4])
def test_single_step_exact_state(torch, orc, gz):
    """One step from exactly the state the GPU holds (no input rounding): velocity,
    density and order parameter agree to FP32 round-off of the step itself."""
    prob = _periodic_random_problem(16, 12, 10, g=(1e-4, -2e-4, gz))
    p, fr, fb, h = random_state(orc, prob, seed=5)
    st, _, _ = state_to_f32(fr, fb)
    sim = _sim(prob)
    sim.set_state(torch.from_numpy(st).cuda(), t=0)
    fr64, fb64 = _internal_state(sim, prob)
    sim.step(1)
    orc.step(p, prob.A, fr64, fb64, np.zeros((2 * Q, p.nx * p.ny)), 0, 1)
    fo = oracle_fields(orc, p, fr64, fb64)
    fg = gpu_fields(sim)
    errs = {k: rel_linf(fg[k], fo[k]) for k in ("rho", "u", "phi", "rho_r")}
    say(f"  exact-state g_z={gz}: rel Linf {errs}")
    for k, tol in (("rho", 1e-6), ("u", 1e-6), ("phi", 2e-6), ("rho_r", 2e-6)):
        assert errs[k] < tol, k


def test_droplet_init_matches(torch, orc):
    prob = droplet_small()
    sim = _sim(prob)
    p, fr, fb, h = oracle_init(orc, prob)
    gr, gb = _gpu_state(sim)
    assert np.abs(gr - fr).max() < 1e-6 and np.abs(gb - fb).max() < 1e-6


# rel L-inf bars after 200 steps.  The 32^3 droplet (tau = 1) carries the
# stated 1e-5 on density and velocity.  Its tau != 1, gamma = 2, gravity
# variant (not a stated configuration) exercises the central-moment
# relaxation at tau ~ 0.53, where the non-equilibrium stress is nearly
# reflected every step and FP32 rounding accumulates; its velocity bar lies
# between the two floors test_oracle_storage_floor measures on the CPU: FP32
# storage with exact arithmetic (DROPLET_CM_U_FLOOR = 2.8e-6) and the plain
# FP32 scheme (DROPLET_CM_U_PLAIN_FP32 = 1.9e-4).  MI355X measures 2.8e-5.
BARS = {"droplet-32": {"rho": 1e-5, "u": 1e-5, "phi": 1e-5, "rho_r": 1e-5},
        "droplet-32-cm": {"rho": 1e-5, "u": 5e-5, "phi": 1e-5, "rho_r": 1e-5}}


@pytest.mark.parametrize("mk", [droplet_small, droplet_cm])
def test_droplet_200_steps(torch, orc, mk):
    """The 32^3 droplet (tau = 1) and its tau != 1, gamma = 2, gravity variant
    after 200 steps against the oracle."""
    prob = mk()
    say(f"droplet {prob.name} {prob.steps} steps")
    sim = _sim(prob)
    sim.step(prob.steps)
    fg = gpu_fields(sim)
    p, fr, fb, h = oracle_init(orc, prob)
    orc.step(p, prob.A, fr, fb, h, 0, prob.steps)
    fo = oracle_fields(orc, p, fr, fb)
    errs = {k: rel_linf(fg[k], fo[k]) for k in ("rho", "u", "phi", "rho_r")}
    for k, e in errs.items():
        say(f"  {k} rel Linf {e:.3e}  (max |{k}| = {np.abs(fo[k]).max():.3e})")
    for k, e in errs.items():
        assert e <= BARS[prob.name][k], k
    _audit_matches_oracle(sim, fo)


def _audit_matches_oracle(sim, fo):
    """The five FP64 totals of lbm_macroscopic (sum rho_r, sum rho_b, sum rho u
    with the half-force term of Eq. Momentum) against the oracle's sums of the
    same fields: masses to 1e-6 relative (MI355X: up to 1.7e-7 after 200
    droplet steps), momenta to 1e-5 of sum rho |u|."""
    a = sim.macroscopic(audit=True)["audit"]
    rho = fo["rho_r"] + fo["rho_b"]
    ref = [fo["rho_r"].sum(), fo["rho_b"].sum(), *(rho[:, None] * fo["u"]).sum(axis=0)]
    mscale = float((rho * np.linalg.norm(fo["u"], axis=1)).sum())
    say(f"  audit {a} oracle {ref}")
    for k in (0, 1):
        assert abs(a[k] - ref[k]) <= 1e-6 * ref[k], (k, a[k], ref[k])
    for k in (2, 3, 4):
        assert abs(a[k] - ref[k]) <= 1e-5 * mscale, (k, a[k], ref[k], mscale)


def test_periodic_audit_conserves(torch):
    """FP64 audit: per-colour mass and momentum conserved on a periodic box with
    g = 0.  MI355X measures, over 100 steps, red 5.1e-9 and blue 1.4e-9
    relative and momentum 2.5e-7 absolute (bit for bit the same with the
    previous kernels); the bars leave a margin of 3 to 7.  The masses move
    by the FP32 rounding of the stored deviations and colour fractions."""
    prob = droplet_cm().replace(g=(0.0, 0.0, 0.0))
    sim = _sim(prob)
    a0 = sim.macroscopic(audit=True)["audit"]
    sim.step(100)
    a1 = sim.macroscopic(audit=True)["audit"]
    say(f"audit {a0} -> {a1}: red {abs(a1[0] - a0[0]) / a0[0]:.2e}, blue {abs(a1[1] - a0[1]) / a0[1]:.2e}, "
        f"momentum {max(abs(a1[k] - a0[k]) for k in (2, 3, 4)):.2e}")
    assert abs(a1[0] - a0[0]) < 2e-8 * a0[0]
    assert abs(a1[1] - a0[1]) < 1e-8 * a0[1]
    assert max(abs(a1[k] - a0[k]) for k in (2, 3, 4)) < 1e-6


def test_nonfinite_state_is_reported(torch, orc):
    """A NaN population (through lbm_set_state) makes lbm_macroscopic's audit
    return LBM_ERR_NONFINITE instead of totals; a finite state does not."""
    from paper_1804_08923_amd.lbm import LbmError
    prob = _periodic_random_problem(9, 7, 5)
    p, fr, fb, h = random_state(orc, prob, seed=4)
    st, _, _ = state_to_f32(fr, fb)
    sim = _sim(prob)
    sim.set_state(torch.from_numpy(st).cuda(), t=0)
    assert all(np.isfinite(sim.macroscopic(audit=True)["audit"]))
    st[5, 77] = np.nan
    sim.set_state(torch.from_numpy(st).cuda(), t=0)
    with pytest.raises(LbmError) as ei:
        sim.macroscopic(audit=True)
    assert ei.value.code == -4
    sim.close()


def _small_jet(**kw):
    from paper_1804_08923_amd.workloads import jet_problem
    prob = jet_problem("jet-small", 20, 18, 40, D=8, u=0.04, gamma=2.0, eta=1.0, Re=40.0, We=20.0,
                       Fr=2.0, steps=150, noise_amp=0.01, noise_seed=7)
    return prob.replace(**kw)


@pytest.mark.parametrize("steps", [1, 150])
def test_small_jet(torch, orc, steps):
    """Jet boundaries (inflow ghost with seeded noise, free-slip walls,
    convective outflow) and buoyancy on a 20x18x40 lattice."""
    prob = _small_jet()
    say(f"small jet {steps} steps")
    sim = _sim(prob)
    sim.step(steps)
    fg = gpu_fields(sim)
    p, fr, fb, h = oracle_init(orc, prob)
    orc.step(p, prob.A, fr, fb, h, 0, steps)
    fo = oracle_fields(orc, p, fr, fb)
    errs = {k: rel_linf(fg[k], fo[k]) for k in ("rho", "u", "phi", "rho_r")}
    say(f"  rel Linf {errs}")
    for k, e in errs.items():
        assert e <= 1e-5, k
    _audit_matches_oracle(sim, fo)
    gr, gb = _gpu_state(sim)
    scale = np.abs(fr + fb).max()
    assert np.abs(gr - fr).max() / scale < 1e-5
    assert np.abs(gb - fb).max() / scale < 1e-5


@pytest.mark.parametrize("shape,D", [((3, 3, 3), 2.0), ((130, 5, 4), 3.0), ((130, 16, 6), 5.0)])
def test_tiny_jets(torch, orc, shape, D):
    """The jet boundaries where almost every node is next to a wall, the inlet
    or the outlet (the 3x3x3 minimum), and on a row two nodes wider than two
    64-node tiles (at 130x16 12 tiles per plane, in bands for the XCDs): 30
    steps against the oracle."""
    from paper_1804_08923_amd.workloads import jet_problem
    prob = jet_problem("jet-tiny", *shape, D=D, u=0.04, gamma=2.0, eta=1.0, Re=20.0, We=10.0, Fr=2.0,
                       steps=30, noise_amp=0.01, noise_seed=5)
    say(f"tiny jet {shape} D={D}")
    sim = _sim(prob)
    sim.step(prob.steps)
    gr, gb = _gpu_state(sim)
    sim.close()
    p, fr, fb, h = oracle_init(orc, prob)
    orc.step(p, prob.A, fr, fb, h, 0, prob.steps)
    scale = np.abs(fr + fb).max()
    err = max(np.abs(gr - fr).max(), np.abs(gb - fb).max()) / scale
    say(f"  max pop err {err:.2e}")
    assert err < 1e-5

"""The solve that is resident on the chip (one workgroup per box of nodes)
against the tick-by-tick march and the CPU oracle: meshes whose boxes have
remainders along each axis, one box, elongated ones, the largest that fit and
one that does not; every charge model; the initial guess, the limits, and the
march after a wait that ran out.

Tolerances: converged potentials 1e-9 relative against the oracle at
newton_atol 1e-10; 1e-12 between two GPU paths of different summation order at
newton_atol 2e-12, near the FP64 floor of ||F|| (meshes of up to 20,000 nodes;
larger ones are compared at 1e-10 and 1e-9)."""
import numpy as np
import pytest

import synth
from oracle import solver
from paper_1403_7561_amd import qe
from tests import gpu_support as gs
from tests.test_gpu_full_charge import CASES as FULL_CHARGE

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VOLTS = np.array([1.6, 1.5, 0.5, 0.8, 0.4])


def solve(dev, phi=None, check=True, **opts):
    start = None if phi is None else phi.clone()
    out, _, rep = qe.qe_solve(qe.Problem(dev), opts=qe.qe_default_options(**opts), phi=start, check=check)
    return out, rep


def march(monkeypatch, dev, phi=None, check=True, **opts):
    monkeypatch.setenv("QE_RESIDENT", "0")
    try:
        return solve(dev, phi, check, **opts)
    finally:
        monkeypatch.delenv("QE_RESIDENT")


def rel_max(a, b):
    a, b = a.cpu().numpy(), b.cpu().numpy() if torch.is_tensor(b) else b
    return float(np.abs(a - b).max() / np.abs(b).max())


@pytest.mark.parametrize("nx,ny,nz,stat", [
    (9, 9, 9, "fd"), (17, 17, 9, "tf"), (18, 7, 12, "fd"), (5, 33, 11, "mb"), (41, 6, 30, "fd"),
    (32, 24, 24, "fd")])
def test_small_meshes(monkeypatch, nx, ny, nz, stat):
    dev = synth.double_dot_device("r", nx, ny, nz, VOLTS, stat=stat, T_K=300.0 if stat == "mb" else 4.0)
    phi, rep = solve(dev, newton_atol=2e-12)
    ref, rref = march(monkeypatch, dev, newton_atol=2e-12)
    assert rep["res_final"] <= 2e-12 and abs(rep["newton_iters"] - rref["newton_iters"]) <= 1
    assert rel_max(phi, ref) <= 1e-12
    again, _ = solve(dev, newton_atol=2e-12)
    assert torch.equal(phi, again)
    if nx * ny * nz <= 4000:
        _, res = solver.solve(dev, atol=1e-10)
        assert rel_max(phi, res.phi) < 1e-9


@pytest.mark.parametrize("nx,ny,nz", [(13, 11, 101), (49, 47, 33), (65, 65, 33), (81, 64, 41), (248, 32, 31),
                                      (31, 32, 241)])
def test_large_meshes(monkeypatch, nx, ny, nz):
    """An elongated mesh (its thin elements put the floor of ||F|| at 1e-11),
    and up to a little under the V-cycle's smallest mesh of 250,000 nodes; some
    of these have no cut into 256 boxes that fit, which is the march's"""
    dev = synth.double_dot_device("r", nx, ny, nz, VOLTS)
    phi, rep = solve(dev, newton_atol=1e-10)
    ref, _ = march(monkeypatch, dev, newton_atol=1e-10)
    assert rep["res_final"] <= 1e-10
    assert rel_max(phi, ref) <= 1e-9


@pytest.mark.parametrize("name", sorted(FULL_CHARGE))
def test_charge_models(monkeypatch, name):
    dev = FULL_CHARGE[name]()
    phi, _ = solve(dev, newton_atol=1e-10)
    ref, _ = march(monkeypatch, dev, newton_atol=1e-10)
    assert rel_max(phi, ref) <= 1e-9


def test_initial_guess_and_limits(monkeypatch):
    dev = gs.ragged_device()
    ref, _ = march(monkeypatch, dev, newton_atol=2e-12)
    noise = np.random.default_rng(2).standard_normal(ref.numel())
    start = ref + 0.01 * torch.as_tensor(noise, device="cuda")
    phi, rep = solve(dev, start, newton_atol=2e-12, init_guess=1)
    assert rep["init_krylov_iters"] == 0 and rel_max(phi, ref) <= 1e-12
    for opts in (dict(newton_maxit=2), dict(newton_maxit=1, ls_max_halvings=0), dict(krylov_maxit=3, newton_maxit=4)):
        _, a = solve(dev, check=False, newton_atol=2e-12, **opts)
        _, b = march(monkeypatch, dev, check=False, newton_atol=2e-12, **opts)
        for key in ("status", "newton_iters", "n_residual_evals", "ls_halvings"):
            assert a[key] == b[key], (opts, key)
        # the two CG recurrences round differently: one iteration per solve
        assert abs(a["krylov_iters"] - b["krylov_iters"]) <= a["newton_iters"] + 1


@pytest.mark.parametrize("nx,ny,nz", [(17, 17, 9), (33, 29, 41)])
def test_wait_that_runs_out_is_the_march(monkeypatch, nx, ny, nz):
    """a wait limited to one poll gives up; the march then solves the same
    problem from the same start"""
    dev = synth.double_dot_device("r", nx, ny, nz, VOLTS)
    ref, rref = march(monkeypatch, dev, newton_atol=1e-10)
    warm, rwarm = march(monkeypatch, dev, 1.01 * ref, newton_atol=1e-10, init_guess=1)
    monkeypatch.setenv("QE_RESIDENT_POLLS", "1")
    phi, rep = solve(dev, newton_atol=1e-10)
    assert torch.equal(phi, ref) and rep == rref
    phi, rep = solve(dev, 1.01 * ref, newton_atol=1e-10, init_guess=1)
    assert torch.equal(phi, warm) and rep == rwarm


@pytest.mark.parametrize("sizes", [[(9, 9, 9)], [(33, 33, 17), (13, 12, 11), (49, 41, 33), (17, 17, 9), (5, 6, 60)] * 3,
                                   [(31, 32, 241), (17, 17, 9)]])
def test_batch(monkeypatch, sizes):
    """instances of different sizes share the chip; the third batch has one
    that may not fit"""
    devs = [synth.double_dot_device(f"b{k}", *s, VOLTS * (1.0 - 0.02 * k)) for k, s in enumerate(sizes)]
    probs = [qe.Problem(d) for d in devs]
    opts = qe.qe_default_options(newton_atol=1e-10)
    phis, _, reps = qe.qe_solve_batch(probs, opts=opts)
    monkeypatch.setenv("QE_RESIDENT", "0")
    refs, _, _ = qe.qe_solve_batch(probs, opts=opts)
    monkeypatch.delenv("QE_RESIDENT")
    for phi, ref, rep in zip(phis, refs, reps):
        assert rep["status"] == 0 and rep["res_final"] <= 1e-10
        assert rel_max(phi, ref) <= 1e-9
    monkeypatch.setenv("QE_RESIDENT_POLLS", "1")
    late, _, reps = qe.qe_solve_batch(probs, opts=opts)
    for phi, ref, rep in zip(late, refs, reps):
        assert rep["status"] == 0 and rel_max(phi, ref) <= 1e-9

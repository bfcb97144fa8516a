"""The automatic choice between Jacobi and the V-cycle within a solve: a Newton
step's CG that a limited number of Jacobi iterations does not finish is taken
by multigrid, as are the steps after it.  Against the solve with Jacobi alone
and the oracle (potentials to 1e-9 relative, the standing tolerance), with the
size thresholds lowered to meshes that the oracle solves."""
import numpy as np
import pytest

import synth
from oracle import solver
from paper_1403_7561_amd import qe
from tests.test_gpu_full_charge import CASES as FULL_CHARGE

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DEVICES = {
    "stack": lambda: synth.double_dot_device("t", 36, 30, 20, np.array([1.5, 1.4, 0.5, 0.7, 0.3])),
    "junction": FULL_CHARGE["pn_mb300K_complete"],
}


def rel_max(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


@pytest.mark.parametrize("name", sorted(DEVICES))
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("trial", [0, 1, 12, 1000])
def test_trial_then_multigrid(monkeypatch, name, precision, trial):
    monkeypatch.setenv("QE_MG_MIN_NODES", "1000")
    monkeypatch.setenv("QE_MG_MIN_COARSE", "300")
    monkeypatch.setenv("QE_MG_LARGE_NODES", "1000")
    monkeypatch.setenv("QE_MG_TRIAL", str(trial))
    dev = DEVICES[name]()
    P = qe.Problem(dev)
    opts = dict(newton_atol=1e-10, precision=precision)
    phi, _, rep = qe.qe_solve(P, opts=qe.qe_default_options(**opts))
    jac, _, repj = qe.qe_solve(P, opts=qe.qe_default_options(precond=1, **opts))
    assert rep["status"] == 0 and rep["res_final"] <= 1e-10 and rep["mg_levels"] >= 2
    steps = rep["krylov_iters"] - rep["init_krylov_iters"] - rep["mg_krylov_iters"]
    # a trial of one iteration per Newton step until one does not suffice (the
    # junction's first steps, whose charge dominates the diagonal, need no more)
    assert trial != 1 or 1 <= steps <= rep["newton_iters"]
    assert rel_max(phi.cpu().numpy(), jac.cpu().numpy()) <= 1e-9
    if trial == 12 and precision == 0:
        _, res = solver.solve(dev, atol=1e-10)
        assert rel_max(phi.cpu().numpy(), res.phi) <= 1e-9


def test_iteration_limit_below_the_trial(monkeypatch):
    """krylov_maxit at or below the trial's length: no trial, the limit holds"""
    monkeypatch.setenv("QE_MG_MIN_NODES", "1000")
    monkeypatch.setenv("QE_MG_LARGE_NODES", "1000")
    P = qe.Problem(DEVICES["stack"]())
    _, _, rep = qe.qe_solve(P, opts=qe.qe_default_options(newton_atol=1e-10, krylov_maxit=5, newton_maxit=3), check=False)
    assert rep["krylov_iters"] <= 5 * 4

"""Solves that the resident kernel does not finish: they are solved again from
the caller's start, whole, by the march or the host-driven iteration.

Potentials 1e-9 relative at newton_atol 1e-10, the standing tolerance, where
two paths of different summation order are compared."""
import numpy as np
import pytest

import synth
from paper_1403_7561_amd import qe

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VOLTS = np.array([1.6, 1.5, 0.5, 0.8, 0.4])


def rel_max(a, b):
    return float((a - b).abs().max() / b.abs().max())


@pytest.mark.parametrize("polls", ["1", "40", "400"])
def test_batch_with_waits_that_run_out(monkeypatch, polls):
    """instances of one box and of many in a launch whose waits run out at
    different places: no instance is left with a part missing"""
    sizes = [(6, 5, 7), (33, 33, 17), (9, 9, 9), (17, 17, 9)] * 24
    probs = [qe.Problem(synth.double_dot_device(f"f{k}", *s, VOLTS * (1.0 - 0.004 * k))) for k, s in enumerate(sizes)]
    opts = qe.qe_default_options(newton_atol=1e-10)
    monkeypatch.setenv("QE_RESIDENT", "0")
    refs, _, _ = qe.qe_solve_batch(probs, opts=opts)
    monkeypatch.delenv("QE_RESIDENT")
    monkeypatch.setenv("QE_RESIDENT_POLLS", polls)
    for _ in range(3):
        phis, _, reps = qe.qe_solve_batch(probs, opts=opts)
        for phi, ref, rep in zip(phis, refs, reps):
            assert rep["status"] == 0 and rep["res_final"] <= 1e-10 and rel_max(phi, ref) <= 1e-9


@pytest.mark.parametrize("n", [(33, 29, 21), (65, 65, 33)])
def test_start_is_the_callers_whatever_was_written(monkeypatch, n):
    """a warm start whose waits run out anywhere, the last exchange included,
    where some workgroups have finished: the result is bit for bit that of the
    whole resident solve or that of the march from the caller's start.  (One
    short Newton step, so that the last exchange is one of four.)"""
    P = qe.Problem(synth.double_dot_device("w", *n, VOLTS))
    ws = qe.workspace_for(P)
    start = 1.001 * qe.qe_solve(P, ws=ws)[0]
    opts = qe.qe_default_options(newton_atol=1e-10, init_guess=1, newton_maxit=1, krylov_maxit=1, krylov_rtol_max=0.99)

    def step():
        return qe.qe_solve(P, opts=opts, phi=start.clone(), want_density=False, ws=ws, check=False)[0]

    resident = step()
    monkeypatch.setenv("QE_RESIDENT", "0")
    march = step()
    monkeypatch.delenv("QE_RESIDENT")
    seen = [0, 0]
    for k in range(1200):
        monkeypatch.setenv("QE_RESIDENT_POLLS", str(1 + k % 60))
        phi = step()
        which = 0 if torch.equal(phi, resident) else 1
        assert which == 0 or torch.equal(phi, march), k
        seen[which] += 1
    assert seen[1] > 0


def thin():
    """its thin elements put the floor of ||F|| at 1e-11: the line search fails"""
    return synth.double_dot_device("l", 13, 11, 101, VOLTS)


def floating():
    """no Dirichlet node: J is singular for the charge-free guess, and the CG breaks down"""
    dev = synth.double_dot_device("l", 17, 17, 9, VOLTS)
    dev.dir_id[:] = -1
    return dev


@pytest.mark.parametrize("make,status", [(thin, -5), (floating, -6)])
def test_failure_is_the_marchs(monkeypatch, make, status):
    """a line search that fails and a CG that breaks down: the status, the
    report and the last iterate are those of the march, whose CG takes p^T J p
    directly; so with a warm start, and in the batch (which skips a linear
    guess that fails)"""
    P = qe.Problem(make())

    def solves():
        opts = dict(newton_atol=2e-12, newton_maxit=20)
        phi, n, rep = qe.qe_solve(P, opts=qe.qe_default_options(**opts), check=False)
        out = [(phi, n, rep)]
        if status == -5:
            out.append(qe.qe_solve(P, opts=qe.qe_default_options(init_guess=1, **opts), phi=0.9 * phi, check=False))
        phis, _, reps = qe.qe_solve_batch([P, P], opts=qe.qe_default_options(**opts), check=False)
        return out + [(f, f, rep) for f, rep in zip(phis, reps)]

    got = solves()
    monkeypatch.setenv("QE_RESIDENT", "0")
    ref = solves()
    assert ref[0][2]["status"] == status
    for (phi, n, rep), (rphi, rn, rrep) in zip(got, ref):
        assert rep == rrep
        if rrep["status"] in (-5, -6):
            assert torch.equal(phi, rphi) and torch.equal(n, rn)

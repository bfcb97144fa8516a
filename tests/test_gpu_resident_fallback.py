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

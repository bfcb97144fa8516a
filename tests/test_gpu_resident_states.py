"""The resident solve with eigenstates' electrons against the host-driven solve
and the oracle: 3D and 1D confinement, a quantum region, full charge; more
states than one and the most that are allowed, supports that miss the mesh's
corner boxes and that cover all of it; the initial guess, and the host-driven
solve after a wait that ran out.  Potentials 1e-9 relative at newton_atol 1e-10,
the standing tolerance."""
import numpy as np
import pytest

import synth
from oracle import solver
from paper_1403_7561_amd import qe
from tests.test_gpu_quantum import CASES, pc_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def everywhere(n, conf=3):
    """n states that are nowhere zero, levels on both sides of the Fermi level"""
    dev = pc_device(2, conf)
    rng = np.random.default_rng(n)
    N = dev.nx * dev.ny * dev.nz
    psi2 = 1e-5 * (0.1 + rng.random((n, N)))
    q = dev.quantum
    dev.quantum = synth.QuantumStates(psi2=psi2, phi_k=q.phi_k, E_i=np.linspace(-0.004, 0.004, n), confinement=q.confinement)
    return dev


DEVICES = {**CASES, "one_everywhere": lambda: everywhere(1), "most_everywhere": lambda: everywhere(32),
           "1d_everywhere": lambda: everywhere(3, 1)}


def solve(P, phi=None, **opts):
    out, _, rep = qe.qe_solve(P, opts=qe.qe_default_options(newton_atol=1e-10, **opts),
                              phi=None if phi is None else phi.clone())
    return out, rep


def rel_max(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


@pytest.mark.parametrize("name", sorted(DEVICES))
def test_resident_states(monkeypatch, name):
    dev = DEVICES[name]()
    P = qe.Problem(dev)
    phi, rep = solve(P)
    again, _ = solve(P)
    assert torch.equal(phi, again)
    monkeypatch.setenv("QE_RESIDENT", "0")
    host, rhost = solve(P)
    warm_start = host + 0.002
    warm_host, _ = solve(P, warm_start, init_guess=1)
    monkeypatch.delenv("QE_RESIDENT")
    assert rep["res_final"] <= 1e-10 and abs(rep["newton_iters"] - rhost["newton_iters"]) <= 1
    assert rel_max(phi.cpu().numpy(), host.cpu().numpy()) <= 1e-9
    warm, _ = solve(P, warm_start, init_guess=1)
    assert rel_max(warm.cpu().numpy(), warm_host.cpu().numpy()) <= 1e-9
    monkeypatch.setenv("QE_RESIDENT_POLLS", "1")
    late, rlate = solve(P)
    assert torch.equal(late, host) and rlate == rhost
    _, res = solver.solve(dev, atol=1e-10)
    assert rel_max(phi.cpu().numpy(), res.phi) <= 1e-9

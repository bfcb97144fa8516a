"""Which solves run resident on the chip: the shapes that have a cut do, the
others do not, and a wait that runs out is seen (qe_last_routes; 0: solved
otherwise, 1: resident, 2: tried resident and solved otherwise)."""
import numpy as np
import pytest

import synth
from paper_1403_7561_amd import qe
from tests.test_gpu_quantum import CASES as STATES

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VOLTS = np.array([1.6, 1.5, 0.5, 0.8, 0.4])
OTHER, RESIDENT, LEFT = 0, 1, 2


def routes(n=64):
    out = (qe.ctypes.c_uint8 * n)()
    k = qe.load_library().qe_last_routes(out, n)
    return list(out)[:k]


def problem(nx, ny, nz, k=0):
    return qe.Problem(synth.double_dot_device("r", nx, ny, nz, VOLTS * (1.0 - 0.01 * k)))


def solve(P, **opts):
    phi, _, rep = qe.qe_solve(P, opts=qe.qe_default_options(newton_atol=1e-9, **opts))
    return phi, routes()


PLATE = (330, 250, 3)   # boxes of 16x16x3 nodes at most: 336 of them


# meshes of up to 250,000 nodes, unless they are plates or needles
@pytest.mark.parametrize("size", [(2, 2, 3), (9, 9, 9), (17, 17, 9), (18, 7, 12), (41, 6, 30), (13, 11, 101), (32, 24, 24),
                                  (65, 65, 33), (81, 64, 41), (248, 32, 31), (31, 32, 241), (63, 63, 62)])
def test_meshes_that_fit(monkeypatch, size):
    P = problem(*size)
    phi, r = solve(P)
    assert r == [RESIDENT]
    _, r = solve(P, init_guess=1)
    assert r == [RESIDENT]
    out = torch.zeros(P.N, dtype=torch.float64, device="cuda")
    qe.qe_solve_static(P, out, opts=qe.qe_default_options(newton_atol=1e-9))
    assert routes() == [RESIDENT] and torch.equal(out, phi)
    monkeypatch.setenv("QE_RESIDENT_POLLS", "1")
    assert solve(P)[1] == [LEFT]
    monkeypatch.setenv("QE_RESIDENT", "0")
    assert solve(P)[1] == [OTHER]


def test_solves_of_other_kinds():
    assert solve(problem(*PLATE))[1] == [OTHER]
    assert solve(problem(17, 17, 9), precision=1)[1] == [OTHER]
    stack = problem(129, 129, 65)
    assert solve(stack)[1] == [RESIDENT, OTHER]             # the coarse start, then the V-cycle's solve
    assert solve(stack, precond=1)[1] == [RESIDENT, OTHER]
    assert solve(stack, precond=1, init_guess=0)[1] == [OTHER]


@pytest.mark.parametrize("name", sorted(STATES))
def test_states(monkeypatch, name):
    P = qe.Problem(STATES[name]())
    assert solve(P)[1] == [RESIDENT]
    monkeypatch.setenv("QE_RESIDENT_POLLS", "1")
    assert solve(P)[1] == [LEFT]


def test_batches(monkeypatch):
    small, large = [problem(33, 33, 17, k) for k in range(40)], [problem(65, 65, 33, k) for k in range(8)]
    opts = qe.qe_default_options(newton_atol=1e-9)
    qe.qe_solve_batch(small, opts=opts)
    assert routes() == [RESIDENT] * 40
    qe.qe_solve_batch(large, opts=opts)                     # marched together: 20 against 30 ms
    assert routes() == [OTHER] * 8
    mixed = [problem(17, 17, 9, k) for k in range(12)] + [problem(*PLATE)]
    qe.qe_solve_batch(mixed, opts=opts)
    assert routes() == [OTHER] * 13                         # the plate has no cut; beside its march the small ones cost little
    monkeypatch.setenv("QE_RESIDENT_POLLS", "1")
    qe.qe_solve_batch(small, opts=opts)
    r = routes()
    assert len(r) == 40 and OTHER not in r and LEFT in r
    monkeypatch.setenv("QE_RESIDENT", "0")
    qe.qe_solve_batch(small, opts=opts)
    assert routes() == [OTHER] * 40

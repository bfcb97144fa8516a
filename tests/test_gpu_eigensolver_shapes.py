"""The eigensolver's Chebyshev preconditioner where its eigenvalue bound and
its pairing of columns can go wrong: one column, odd and even numbers of them,
the most that are allowed; spacings with aspect ratios up to 50, per-axis
masses, steps of several eV and potentials that vary within an element.
Tolerances of the eigensolver's other tests (levels 1e-9 relative, states
1e-8)."""
import numpy as np
import pytest

from tests.test_gpu_schrodinger import compare, mesh_problem

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")


@pytest.mark.parametrize("n,dims,stretch,step", [
    (1, (3, 4, 9), 1.0, 0.0), (2, (9, 8, 7), 1.3, 5.0), (7, (12, 11, 10), 1.5, 0.0), (5, (8, 15, 16), 1.2, 3.1),
    (16, (14, 13, 12), 1.0, 1.0)])
def test_shapes_against_the_oracle(n, dims, stretch, step):
    rng = np.random.default_rng(n)
    x, y, z = [np.concatenate([[0.0], np.cumsum(0.4 * s ** np.arange(m - 1))])
               for m, s in zip(dims, (stretch, 1.0, 1.0 / stretch))]
    P = mesh_problem(x, y, z)
    E = int(np.prod(np.array(dims) - 1))
    k, j, i = np.meshgrid(*[np.arange(m) for m in dims[::-1]], indexing="ij")
    fixed = ((k == 0) | (j == dims[1] - 1)).ravel()
    upper = np.repeat(np.arange(dims[2] - 1) >= (dims[2] - 1) // 2, (dims[0] - 1) * (dims[1] - 1))
    masses = 1.0 / np.stack([np.full(E, 0.19), np.full(E, 0.3), np.full(E, 0.98)]) * (1.0 + 0.1 * rng.random((3, E)))
    compare(P, masses, np.where(upper, step, 0.0), 0.3 * rng.standard_normal(P.N), fixed, n)

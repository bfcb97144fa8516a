"""Electron counts over the index ranges of their boxes: boxes that hold no
element, one, a slab, everything, that overlap and that lie apart, on meshes with
a remainder in every direction.  1e-10 relative to the oracle's sum over the same
elements (sums of at most 10^4 terms of one sign: rounding below 1e-12)."""
import numpy as np
import pytest

import synth
from oracle import solver
from paper_1403_7561_amd import qe

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

INF = float("inf")
BOXES = {
    "none": [(500.0, 600.0, 0.0, 10.0, 0.0, 10.0)],
    "between_centres": [(0.0, 0.01, 0.0, 0.01, 0.0, 0.01)],
    "everything": [(-INF, INF, -INF, INF, -INF, INF)],
    "slab": [(-INF, INF, 60.0, 140.0, 80.0, 95.0)],
    "apart_and_overlapping": [(0.0, 40.0, 0.0, 200.0, 60.0, 90.0), (160.0, 200.0, 0.0, 90.0, 0.0, 100.0),
                              (20.0, 180.0, 50.0, 60.0, 10.0, 99.0), (500.0, 600.0, 0.0, 1.0, 0.0, 1.0)],
}


@pytest.mark.parametrize("name", sorted(BOXES))
@pytest.mark.parametrize("dims", [(7, 9, 8), (33, 20, 17)])
def test_counts(name, dims):
    dev = synth.double_dot_device("c", *dims, np.array([1.6, 1.5, 0.5, 0.8, 0.4]))
    po = solver.make_problem(dev)
    phi = 0.45 + 0.2 * np.random.default_rng(1).random(np.prod(dims))
    got = qe.qe_count_electrons(qe.Problem(dev), torch.as_tensor(phi, device="cuda"), BOXES[name])
    want = np.array([po.count(phi, b) for b in BOXES[name]])
    assert np.allclose(got, want, rtol=1e-10, atol=0.0)

"""Calls of several host threads at once, a stream and a workspace each: solves
that want the whole chip take turns or march, and none stalls another.

Potentials 1e-9 relative against the same calls one after the other at
newton_atol 1e-10, the standing tolerance between two paths; the time is bounded
by a hundred times what the calls take one after the other (a wait that has to
run out takes seconds, the calls milliseconds)."""
import threading
import time

import numpy as np
import pytest

import synth
from paper_1403_7561_amd import qe

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VOLTS = np.array([1.6, 1.5, 0.5, 0.8, 0.4])


def device(k, size):
    return synth.double_dot_device(f"c{k}", *size, VOLTS * (1.0 - 0.01 * k))


def single(k, size):
    """five solves, cold and warm in turn"""
    P, opts = qe.Problem(device(k, size)), qe.qe_default_options(newton_atol=1e-10)
    ws = qe.workspace_for(P, opts)

    def run():
        out, phi = [], None
        for i in range(5):
            opts.init_guess = 1 if i % 2 else 2
            phi, _, _ = qe.qe_solve(P, opts=opts, phi=1.01 * phi if i % 2 else None, ws=ws)
            out.append(phi)
        return out
    return run


def batch(k, size, n):
    probs, opts = [qe.Problem(device(k + i, size)) for i in range(n)], qe.qe_default_options(newton_atol=1e-10)
    ws = qe.Workspace(qe.qe_batch_workspace_bytes(probs, opts), probs[0].device)
    return lambda: qe.qe_solve_batch(probs, opts=opts, ws=ws)[0]


JOBS = {
    "solves": lambda: [single(k, (65, 65, 33)) for k in range(2)],
    "batches": lambda: [batch(10 * k, (33, 33, 17), 40) for k in range(2)],
    "both": lambda: [single(0, (65, 65, 33)), batch(1, (33, 33, 17), 40), single(3, (17, 17, 9)), batch(5, (65, 65, 33), 8)],
}


@pytest.mark.parametrize("name", sorted(JOBS))
def test_threads(name):
    jobs = JOBS[name]()
    t = time.time()
    refs = [job() for job in jobs]
    torch.cuda.synchronize()
    alone = time.time() - t
    out, errors = [None] * len(jobs), []
    gate = threading.Barrier(len(jobs))

    def body(i, stream):
        try:
            with torch.cuda.stream(stream):
                gate.wait()
                out[i] = jobs[i]()
                stream.synchronize()
        except BaseException as e:   # noqa: B902 (reported by the test's own thread)
            errors.append(e)

    for _ in range(5):
        threads = [threading.Thread(target=body, args=(i, torch.cuda.Stream())) for i in range(len(jobs))]
        t = time.time()
        for th in threads:
            th.start()
        for th in threads:
            th.join()
        assert not errors and time.time() - t < 100.0 * alone
        for got, ref in zip(out, refs):
            for phi, r in zip(got, ref):
                assert float((phi - r).abs().max()) <= 1e-9 * float(r.abs().max())

"""Solves in one launch, whose workgroups wait for each other inside the kernel, against the same solve with a launch per round."""
import threading

import numpy as np
import pytest

import paper_2008_03433_amd as tron
from datagen import DenseProblem
from oracle import LOSS_LR, LOSS_L2SVM
from util import torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture
def knob():
    def set_to(name, value):
        tron.tron_tuning_set(name, value)
        used.add(name)
    used = set()
    yield set_to
    for name in used:
        tron.tron_tuning_set(name, -1)


def _dense(rng, n, d):
    X = rng.standard_normal((n, d))
    y = np.where(X @ rng.standard_normal(d) + rng.standard_normal(n) > 0.0, 1.0, -1.0)
    return DenseProblem("resident", n, d, X, y)


def _solve(ds, loss, C, w0, **kw):
    w = w0.clone()
    r = ds.solve(loss, C, 1e-4, w, **kw)
    return w.cpu().numpy().tobytes(), r.f, r.gnorm, r.outer_iters, r.cg_iters_total, r.status, r.trace


# one to four lanes per row, several tiles at a time up to four columns; one workgroup, one counter (up to 64 workgroups of 512
# rows) and eight, one tile per wavefront (up to 131,072 rows) and more
@pytest.mark.parametrize("loss", [LOSS_LR, LOSS_L2SVM])
@pytest.mark.parametrize("n,d", [(1, 3), (700, 24), (32_768, 12), (32_769, 12), (131_072, 7), (131_073, 30), (300_007, 4), (300_007, 1)])
def test_dense_solve_in_one_launch_has_the_bits_of_a_launch_per_round(rng, knob, loss, n, d):
    torch = torch_mod()
    ds = tron.Dataset.from_problem(_dense(rng, n, d))
    w0 = torch.zeros(d, dtype=torch.float64, device="cuda")
    try:
        for start in (w0, w0 + 0.1):
            one = _solve(ds, loss, 0.3, start)
            assert _solve(ds, loss, 0.3, start) == one
            knob("solve_wait_us", 0)    # every workgroup gives up at once, the solve starts again with a launch per round
            assert _solve(ds, loss, 0.3, start) == one
            knob("solve_wait_us", -1)
            knob("solve_resident", 0)
            assert _solve(ds, loss, 0.3, start) == one
            knob("solve_resident", -1)
            assert _solve(ds, loss, 0.3, start) == one
    finally:
        ds.close()


def test_solves_of_several_threads_on_streams_of_their_own(rng):
    """More workgroups in all than the GPU has compute units: the solves take turns, with the results they have alone."""
    torch = torch_mod()
    problems = [_dense(rng, n, 24) for n in (90_000, 131_072, 20_000, 131_073)]
    alone, together = {}, {}

    def work(k, out):
        with torch.cuda.stream(torch.cuda.Stream()):
            ds = tron.Dataset.from_problem(problems[k])
            w0 = torch.zeros(24, dtype=torch.float64, device="cuda")
            out[k] = [_solve(ds, LOSS_L2SVM, 0.3, w0) for _ in range(5)]
            ds.close()

    for k in range(len(problems)):
        work(k, alone)
    threads = [threading.Thread(target=work, args=(k, together)) for k in range(len(problems))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert together == alone

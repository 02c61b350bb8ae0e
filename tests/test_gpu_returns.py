"""What a call returns is there when it returns: read at once on another stream than the handle's, and by the host, without a wait
for the handle's stream."""
import numpy as np
import pytest

import paper_2008_03433_amd as tron
from datagen import DenseProblem, SparseProblem
from oracle import LOSS_LR, LOSS_L2SVM, Oracle
from util import torch_mod

pytestmark = pytest.mark.gpu


def _dense(rng, n, d):
    X = rng.standard_normal((n, d))
    return DenseProblem("returns", n, d, X, np.where(X @ rng.standard_normal(d) > 0.0, 1.0, -1.0))


def _sparse(rng, n, d, mean):
    rows = rng.integers(1, 2 * mean, n)
    col = np.concatenate([np.sort(rng.choice(d, k, replace=False)) for k in rows]).astype(np.int32)
    return SparseProblem("returns", n, d, np.concatenate([[0], np.cumsum(rows)]).astype(np.int64), col, rng.standard_normal(col.size) / np.sqrt(mean),
                         np.where(rng.random(n) < 0.5, 1.0, -1.0))


# the pass's last workgroup forms the results, or a second launch over the columns does; sparse: the product's own launch (whose
# other workgroups may still be writing: the call waits for the stream), or one that adds up the sums of many workgroups
PROBLEMS = {"dense": lambda rng: _dense(rng, 5003, 24), "dense_one": lambda rng: _dense(rng, 1, 1), "dense_wide": lambda rng: _dense(rng, 3001, 257),
            "sparse": lambda rng: _sparse(rng, 1500, 900, 12), "sparse_long": lambda rng: _sparse(rng, 2000, 600_000, 40)}


@pytest.mark.parametrize("loss", [LOSS_LR, LOSS_L2SVM])
@pytest.mark.parametrize("name", PROBLEMS)
def test_products_are_there_on_another_stream(rng, loss, name):
    torch = torch_mod()
    p = PROBLEMS[name](rng)
    o = Oracle.from_problem(p)
    other = torch.cuda.Stream()
    ds = tron.Dataset.from_problem(p)
    try:
        for k in range(6):
            w, v = 0.3 * rng.standard_normal(p.d), rng.standard_normal(p.d)
            wd, vd = torch.from_numpy(w).cuda(), torch.from_numpy(v).cuda()
            g, Hv = torch.zeros_like(wd), torch.zeros_like(wd)
            torch.cuda.synchronize()
            f = ds.fun_grad(loss, 0.7, wd, g)
            with torch.cuda.stream(other):
                g1 = g.clone()
            vHv = ds.hv(0.7, vd, Hv)
            with torch.cuda.stream(other):
                Hv1 = Hv.clone()
            torch.cuda.synchronize()
            f_ref, g_ref, D = o.fun_grad(loss, 0.7, w)
            Hv_ref = o.hv(0.7, D, v)
            for got, ref in ((g1.cpu().numpy(), g_ref), (Hv1.cpu().numpy(), Hv_ref)):   # sums of up to 5003 terms in fp64
                assert np.linalg.norm(got - ref) <= 1e-11 * np.linalg.norm(ref)
            assert abs(f - f_ref) <= 1e-11 * abs(f_ref) and abs(vHv - v @ Hv_ref) <= 1e-11 * abs(v @ Hv_ref)
    finally:
        ds.close()


# rounds of less and of more than 16 MB (two rounds kept enqueued, or one), which are still to run when the solve returns
@pytest.mark.parametrize("n", [700, 120_003])
def test_batch_calls_behind_one_another(rng, n):
    torch = torch_mod()
    p = _dense(rng, n, 20)
    ds = tron.Dataset.from_problem(p)
    other = torch.cuda.Stream()
    K, C = 3, [0.05, 0.1, 0.2]
    batch = tron.Batch(ds, K, torch.from_numpy(rng.integers(0, 1 << K, n, dtype=np.int32)).cuda())
    try:
        def calls(wait):
            out = []
            for k in range(4):
                W = torch.full((K, 20), 0.01 * k, dtype=torch.float64, device="cuda")
                G, HV = torch.zeros_like(W), torch.zeros_like(W)
                torch.cuda.synchronize()
                r = batch.solve(LOSS_L2SVM, C, 1e-3, W)
                with torch.cuda.stream(other):
                    W1 = W.clone()
                if wait:
                    torch.cuda.synchronize()
                f = batch.fun_grad(LOSS_L2SVM, C, W, G)
                with torch.cuda.stream(other):
                    G1 = G.clone()
                if wait:
                    torch.cuda.synchronize()
                c = batch.hv(C, G1, HV)
                with torch.cuda.stream(other):
                    HV1 = HV.clone()
                torch.cuda.synchronize()
                out.append(([x.f for x in r], [x.outer_iters for x in r], [x.trace for x in r], list(f), list(c), [t.cpu().numpy().tobytes() for t in (W1, G1, HV1)]))
            return out

        assert calls(False) == calls(True)
    finally:
        batch.close()
        ds.close()


# the active set as a bit a row and fp64 D; rows in registers, one tile at a time, several (few columns), a launch per round
@pytest.mark.parametrize("loss", [LOSS_LR, LOSS_L2SVM])
@pytest.mark.parametrize("n,d", [(20_000, 24), (400_003, 24), (400_003, 3)])
def test_D_is_there_for_a_captured_product_on_another_stream(loss, n, d):
    """A captured tron_hv_static, replayed on another stream as soon as a call has returned that replaced the D it reads."""
    torch = torch_mod()
    rng = np.random.default_rng(n + d)
    own, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(own):
        ds = tron.Dataset.from_problem(_dense(rng, n, d))
    points = [torch.from_numpy(s * rng.standard_normal(d)).cuda() for s in (0.1, 0.3, 1.0)]
    v, out = torch.from_numpy(rng.standard_normal(d)).cuda(), torch.empty(d, dtype=torch.float64, device="cuda")
    w = torch.zeros_like(v)

    def at(k):   # twice: D goes to the handle's two buffers in turn, and the product reads one of them
        ds.fun_grad(loss, 0.5, points[k - 1])
        ds.fun_grad(loss, 0.5, points[k])

    def solved(resident):
        tron.tron_tuning_set("solve_resident", resident)
        w.zero_()
        torch.cuda.synchronize()
        ds.solve(loss, 0.5, 1e-3, w, max_outer=1)
        tron.tron_tuning_set("solve_resident", -1)

    def product():
        out.zero_()
        torch.cuda.synchronize()
        ds.hv_static(0.5, v, out)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    try:
        for calls in ([lambda k=k: at(k) for k in range(3)], [lambda: solved(-1), lambda: solved(0)]):
            calls[0]()
            product()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=own):
                ds.hv_static(0.5, v, out)
            expected = []
            for call in calls:
                at(0)
                call()
                eager = product()
                graph.replay()
                torch.cuda.synchronize()
                expected.append(out.cpu().numpy())   # (the captured call keeps its grid and its rule for rows outside the active set)
                assert np.linalg.norm(expected[-1] - eager) <= 1e-12 * np.linalg.norm(eager)
            for k in range(30):
                at((k + 1) % 3)
                torch.cuda.synchronize()
                calls[k % len(calls)]()
                with torch.cuda.stream(other):
                    graph.replay()
                torch.cuda.synchronize()
                np.testing.assert_array_equal(out.cpu().numpy(), expected[k % len(calls)])
    finally:
        torch.cuda.synchronize()
        ds.close()

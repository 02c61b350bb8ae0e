"""Rows that a problem has nothing to do with may hold any finite numbers, also such whose squares are none: they change no result of a
batch, whichever kernel runs it, the first row of the matrix among them."""
import numpy as np
import pytest

from util import dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def restore():
    yield
    import paper_2008_03433_amd as tron
    tron.tron_tuning_set("batch_mfma", -1)
    tron.tron_tuning_set("batch_mfma_rows", 0)


def everything(X, y, member, K, loss):
    """Results of the calls and of plain and preconditioned solves, by problem."""
    import paper_2008_03433_amd as tron
    torch = torch_mod()
    ds = tron.Dataset.from_dense(X, y)
    try:
        b = tron.Batch(ds, K, member)
        Cs = [0.1 * (k + 1) for k in range(K)]
        g = torch.Generator().manual_seed(K)
        V = torch.randn(K, X.shape[1], generator=g, dtype=torch.float64).cuda()
        G, HV = torch.empty_like(V), torch.empty_like(V)
        f = b.fun_grad(loss, Cs, 0.01 * V, G)
        vHv = b.hv(Cs, V, HV)
        out = [[f[k], vHv[k], G[k].cpu().numpy(), HV[k].cpu().numpy()] for k in range(K)]
        for blend in (0.0, 0.3):
            W = torch.zeros_like(V)
            r = b.solve(loss, Cs, 1e-3, W, precond_blend=blend, max_outer=20, max_cg=30)
            for k in range(K):
                out[k] += [r[k].f, r[k].cg_iters_total, float(r[k].converged), W[k].cpu().numpy()]
        b.close()
        return out
    finally:
        ds.close()


# (K, batch_mfma, batch_mfma_rows): the vector units, the matrix units with half and whole tiles
KERNELS = [(3, 0, 0), (8, 0, 0), (8, 1, 0), (12, -1, 0), (16, -1, 64)]


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("d", [1, 7, 16, 17, 24, 31, 32])
@pytest.mark.parametrize("loss", [0, 1])
def test_rows_of_others(kernel, d, loss):
    import paper_2008_03433_amd as tron
    rng = np.random.default_rng(d)
    K, units, rows = kernel
    tron.tron_tuning_set("batch_mfma", units)
    tron.tron_tuning_set("batch_mfma_rows", rows)
    n = 64 * 40 + 5
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0)
    X = rng.standard_normal((n, d)) + 0.5 * y[:, None]
    member = np.zeros(n, dtype=np.uint32)
    part = rng.integers(0, 6, n)
    for k in range(K):
        member |= (part != k % 6).astype(np.uint32) << np.uint32(k)
    nobody = np.r_[0, 5, 64:70, 128:192, 200:232, n - 1]
    member[nobody] = 0
    only_first = np.r_[70, 300:303, n - 2]
    member[only_first] = 1
    want = everything(X, y, member, K, loss)
    for k in range(K):
        assert want[k][6] == 1.0 and want[k][10] == 1.0
    # rows of no problem: the same bits
    X2 = X.copy()
    X2[nobody] = np.array([1e300, -1e300])[rng.integers(0, 2, (len(nobody), d))]
    for got, exp in zip(everything(X2, y, member, K, loss), want):
        for a, b in zip(got, exp):
            np.testing.assert_array_equal(a, b)
    # rows of the first problem: every other one's results stay what they are.  (1e160: its products with the other problems' vectors are
    # numbers, its square is none)
    X2[only_first] = 1e160
    for got, exp in list(zip(everything(X2, y, member, K, loss), want))[1:]:
        for a, b in zip(got, exp):
            np.testing.assert_array_equal(a, b)

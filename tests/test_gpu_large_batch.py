"""Several problems over a matrix larger than the cache in front of HBM (288 MB), whose tiles come through LDS: two and four lanes a row, odd and
even numbers of columns, ragged last tiles, up to four problems, more, and so many that the
matrix units take them; rows of no problem count for nothing.  The reference is the same
sum on the GPU in torch, in fp64.  Bound: sums of n terms of size about 1 in any order differ by some sqrt(n) eps = 1e-12 of them at most."""
import pytest

from util import torch_mod

pytestmark = pytest.mark.gpu
REL = 1e-11


# 36 million entries are the first that come this way: at the line and above it; the last tile with one row, all but one, full
@pytest.mark.parametrize("n,d", [(4_000_001, 9), (2_400_063, 15), (2_250_000, 16), (2_250_001, 16), (2_117_648, 17), (2_000_127, 18), (1_500_001, 24),
                                 (1_333_376, 28), (1_250_001, 29), (1_161_345, 31), (1_125_057, 32)])
@pytest.mark.parametrize("K", [2, 7, 12])
def test_large_batch(n, d, K):
    import paper_2008_03433_amd as tron
    torch = torch_mod()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + d + K)
    X = torch.randn(n, d, generator=gen, dtype=torch.float64, device="cuda")
    y = torch.where(torch.rand(n, generator=gen, device="cuda") < 0.5, 1.0, -1.0).to(torch.float64)
    X[:, 0] += y
    X[: n // 3, 1] += 3.0 * y[: n // 3]      # whole tiles leave the active sets at W below
    part = torch.randint(8, (n,), generator=gen, device="cuda", dtype=torch.int32)
    part[n // 2: n // 2 + 6400] = 0          # tiles without a row, tiles with a few
    part[n // 2 + 6400::64][:50] = 1
    part[0] = 0                              # the matrix' first row among them
    member = torch.zeros(n, dtype=torch.int32, device="cuda")
    for k in range(K):
        member |= ((part != 0) & (part != 1 + k % 7)).to(torch.int32) << k
    handle = tron.tron_dataset_create_dense_empty(n, d)
    held = X.clone()
    held[part == 0] = 1e300   # (whose squares are no numbers)
    tron.tron_dataset_write_rows(handle, 0, n, held, y)
    del held
    ds = tron.Dataset(handle)
    try:
        b = tron.Batch(ds, K, member)
        Cs = [0.05 * (k + 1) for k in range(K)]
        W = 0.1 * torch.randn(K, d, generator=gen, dtype=torch.float64, device="cuda")
        W[:, 0] += 0.3
        W[:, 1] += 0.8
        V = torch.randn(K, d, generator=gen, dtype=torch.float64, device="cuda")
        G, HV = torch.empty_like(W), torch.empty_like(W)
        rows = torch.stack([(member >> k & 1).to(torch.float64) for k in range(K)])
        Z, U = W @ X.T, V @ X.T
        for loss in (tron.LOSS_LR, tron.LOSS_L2SVM):
            if loss == tron.LOSS_LR:
                h = torch.sigmoid(y * Z)
                zhat, D, each = (h - 1.0) * y, h * (1.0 - h), torch.nn.functional.softplus(-y * Z)
            else:
                act = (y * Z < 1.0).to(torch.float64)
                zhat, D, each = 2.0 * (Z - y) * act, 2.0 * act, (1.0 - y * Z).clamp(min=0.0) ** 2
            C = torch.tensor(Cs, dtype=torch.float64, device="cuda")
            want_f = 0.5 * (W * W).sum(1) + C * (rows * each).sum(1)
            want_G = W + C[:, None] * ((rows * zhat) @ X)
            want_HV = V + C[:, None] * ((rows * D * U) @ X)
            for _ in range(2):
                f = b.fun_grad(loss, Cs, W, G)
                vHv = b.hv(Cs, V, HV)
                for k in range(K):
                    assert abs(f[k] - float(want_f[k])) <= REL * abs(f[k]), (loss, k)
                    assert float((G[k] - want_G[k]).norm() / want_G[k].norm()) <= REL, (loss, k)
                    assert float((HV[k] - want_HV[k]).norm() / want_HV[k].norm()) <= REL, (loss, k)
                    assert abs(vHv[k] - float(V[k] @ want_HV[k])) <= REL * abs(vHv[k])
            for blend in (0.0, 0.3):   # problems that ask for different things in a round, the Hessian diagonal among them
                Ws = torch.zeros_like(W)
                r = b.solve(loss, Cs, 1e-3, Ws, precond_blend=blend, max_outer=60, max_cg=60)
                b.fun_grad(loss, Cs, torch.zeros_like(W), G)
                g0 = G.norm(dim=1)
                f = b.fun_grad(loss, Cs, Ws, G)
                for k in range(K):
                    assert r[k].converged and abs(f[k] - r[k].f) <= REL * abs(f[k]), (loss, blend, k)
                    assert float(G[k].norm()) <= 1e-3 * float(g0[k]) * (1 + 1e-9), (loss, blend, k)
        b.close()
    finally:
        ds.close()

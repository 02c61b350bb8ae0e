"""Dense matrices larger than the cache in front of HBM (288 MB), which come through LDS or by non-temporal loads: odd and even numbers of
columns for each number of lanes a row, ragged last tiles.  The reference is the same sum on the GPU in torch, in fp64.  Bound: sums of
n terms of size about 1 in any order differ by some sqrt(n) eps = 1e-12 of them at most."""
import pytest

from util import torch_mod

pytestmark = pytest.mark.gpu
REL = 1e-11


def close(got, want, what):
    err = float((got - want).norm() / want.norm())
    assert err <= REL, (what, err)


# two lanes a row, four, and 16 to 64 (d > 64); 36 million entries are the first that come this way: just below, at and above it, the last tile
# with one row, all but one, full
@pytest.mark.parametrize("n,d", [(4_000_001, 9), (3_599_999, 10), (3_600_064, 10), (2_400_063, 15), (2_249_999, 16), (2_250_000, 16), (2_250_001, 16), (2_117_648, 17), (2_000_127, 18),
                                 (1_500_001, 24), (1_333_376, 27), (1_161_345, 31), (1_125_057, 32), (450_001, 80), (360_003, 101), (200_003, 257), (70_400, 512)])
def test_large_dense_calls_and_solve(n, d):
    import paper_2008_03433_amd as tron
    torch = torch_mod()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + d)
    X = torch.randn(n, d, generator=gen, dtype=torch.float64, device="cuda")
    y = torch.where(torch.rand(n, generator=gen, device="cuda") < 0.5, 1.0, -1.0).to(torch.float64)
    X[:, 0] += y
    X[: n // 3, 1] += 3.0 * y[: n // 3]      # whole tiles leave the active set at w below, the rest keeps most of its rows
    w = torch.zeros(d, dtype=torch.float64, device="cuda")
    w[0], w[1] = 0.3, 0.8
    v = torch.randn(d, generator=gen, dtype=torch.float64, device="cuda")
    handle = tron.tron_dataset_create_dense_empty(n, d)
    tron.tron_dataset_write_rows(handle, 0, n, X, y)
    ds = tron.Dataset(handle)
    try:
        z, u = X @ w, X @ v
        for loss in (tron.LOSS_LR, tron.LOSS_L2SVM):
            if loss == tron.LOSS_LR:
                h = torch.sigmoid(y * z)
                zhat, D, f = (h - 1.0) * y, h * (1.0 - h), torch.nn.functional.softplus(-y * z).sum()
            else:
                act = (y * z < 1.0).to(torch.float64)
                zhat, D, f = 2.0 * (z - y) * act, 2.0 * act, ((1.0 - y * z).clamp(min=0.0) ** 2).sum()
            g, Hv, diag = torch.empty_like(w), torch.empty_like(w), torch.empty_like(w)
            got = ds.fun_grad(loss, 0.1, w, g)
            assert abs(got - float(0.5 * w @ w + 0.1 * f)) <= REL * abs(got)
            close(g, w + 0.1 * (X.T @ zhat), "gradient")
            vHv = ds.hv(0.1, v, Hv)
            want = v + 0.1 * (X.T @ (D * u))
            close(Hv, want, "product")
            assert abs(vHv - float(v @ want)) <= REL * abs(vHv)
            ds.hess_diag(0.1, diag)
            close(diag, 1.0 + 0.1 * ((X * X).T @ D), "diagonal")
            ds.hv(0.1, v, Hv)   # again, behind the other calls
            close(Hv, want, "product again")
            if d <= 32:   # a solve in one launch: the gradient at its end, from the calls
                ws = torch.zeros_like(w)
                r = ds.solve(loss, 0.1, 1e-3, ws)
                g0 = torch.empty_like(w)
                ds.fun_grad(loss, 0.1, torch.zeros_like(w), g0)
                f_end = ds.fun_grad(loss, 0.1, ws, g)
                assert r.converged and abs(f_end - r.f) <= REL * abs(r.f)
                assert float(g.norm()) <= 1e-3 * float(g0.norm()) * (1 + 1e-9) and abs(float(g.norm()) - r.gnorm) <= 1e-7 * r.gnorm
    finally:
        ds.close()

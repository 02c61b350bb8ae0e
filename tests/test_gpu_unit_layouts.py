"""Layouts without values at the edges of their pieces: transposed products of binary matrices whose sums are whole numbers, so that
every order of summation gives the same bits."""
import numpy as np
import pytest

from util import dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture
def force_partitions():
    import paper_2008_03433_amd as tron
    tron.tron_tuning_set("csr_parts", 8)
    yield
    tron.tron_tuning_set("csr_parts", 0)


def binary_csr(n, d, columns):
    """columns: {feature: instances}."""
    keys = np.unique(np.concatenate([np.asarray(rows, dtype=np.int64) * d + j for j, rows in columns.items()]))
    rows, cols = keys // d, (keys % d).astype(np.int32)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=n), out=rowptr[1:])
    return rowptr, cols


def gradient_at_zero(ds, d):
    """L2-SVM at w = 0: every row is active and zhat = -2 y, so the gradient is -2 C X^T y."""
    import paper_2008_03433_amd as tron
    torch = torch_mod()
    w, g = torch.zeros(d, dtype=torch.float64, device="cuda"), torch.empty(d, dtype=torch.float64, device="cuda")
    ds.fun_grad(tron.LOSS_L2SVM, 1.0, w, g)
    return g.cpu().numpy()


# one window of up to 16,384 instances and the first sizes beyond, several with an odd rest, a last window of one or two instances, more
# windows than divide the compute units evenly
@pytest.mark.parametrize("n", [64, 16_384, 16_385, 32_769, 70_001, 131_072 + 1, 300_007])
def test_hot_rows_in_windows(force_partitions, n):
    import paper_2008_03433_amd as tron
    rng = np.random.default_rng(n)
    d = 2600
    columns = {0: np.arange(n), 1: np.arange(0, n, 2), 2: np.arange(n // 2), 3: np.arange(n - min(n, 700), n), 4: np.array([n - 1]), d - 1: np.arange(n)}
    for j, length in ((5, 255), (6, 256), (7, 257), (8, 512), (9, 513), (10, 31), (11, 32), (12, 33)):   # pieces of 256; the fewest entries of a hot row
        columns[j] = np.arange(min(n, length))
    for j in range(20, 2400):   # more than two groups of 1024 slots, features that are no hot rows among them
        columns[j] = rng.choice(n, size=min(n, int(rng.integers(1, 120))), replace=False)
    rowptr, cols = binary_csr(n, d, columns)
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0)
    ds = tron.Dataset.from_csr(n, d, rowptr, cols, np.ones(len(cols)), y)
    try:
        assert tron.tron_dataset_stat(ds.handle, "unit_values") == 1
        hot = tron.tron_dataset_stat(ds.handle, "bwd_tile_nnz")
        assert tron.tron_dataset_stat(ds.handle, "bwd_tile_rows") > 0 and hot + tron.tron_dataset_stat(ds.handle, "bwd_csr_nnz") == len(cols)
        want = np.zeros(d)
        np.add.at(want, cols, -2.0 * np.repeat(y, np.diff(rowptr)))
        for _ in range(2):
            assert np.array_equal(gradient_at_zero(ds, d), want)
        # a product, too: v of small whole numbers, D = 2
        v = rng.integers(-3, 4, size=d).astype(np.float64)
        torch = torch_mod()
        Hv = torch.empty(d, dtype=torch.float64, device="cuda")
        ds.hv(1.0, dev(v), Hv)
        xv = np.zeros(n)
        np.add.at(xv, np.repeat(np.arange(n), np.diff(rowptr)), v[cols])
        want = v.copy()
        np.add.at(want, cols, 2.0 * np.repeat(xv, np.diff(rowptr)))
        assert np.array_equal(Hv.cpu().numpy(), want)
    finally:
        ds.close()

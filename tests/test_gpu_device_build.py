"""Layouts of unpartitioned sparse matrices built on the device against those built on the host: the same layouts, so the same bits in every
result, and the same errors."""
import numpy as np
import pytest

from util import dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def restore():
    yield
    import paper_2008_03433_amd as tron
    tron.tron_tuning_set("csr_device_build", -1)
    tron.tron_tuning_set("csr_segmented", -1)
    tron.tron_tuning_set("csr_parts", 0)


def csr(rng, n, d, counts, popular=0):
    """counts[i] distinct columns in row i; `popular` columns that are in nearly every row."""
    rows = []
    for m in counts:
        c = rng.choice(d, size=min(int(m), d), replace=False)
        if popular and m:
            c = np.concatenate([c, np.arange(popular)[rng.random(popular) < 0.95]])
        rows.append(np.unique(c))
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum([len(r) for r in rows], out=rowptr[1:])
    cols = np.concatenate(rows).astype(np.int32) if rowptr[n] else np.zeros(0, dtype=np.int32)
    return rowptr, cols, rng.standard_normal(len(cols)), np.where(rng.random(n) < 0.5, 1.0, -1.0)


def results(n, d, arrays, on_device):
    import paper_2008_03433_amd as tron
    torch = torch_mod()
    ds = tron.Dataset.from_csr(n, d, *([dev(a) for a in arrays] if on_device else arrays))
    try:
        g = torch.Generator().manual_seed(1)
        w, v = (0.1 * torch.randn(d, generator=g, dtype=torch.float64)).cuda(), torch.randn(d, generator=g, dtype=torch.float64).cuda()
        out = [tron.tron_dataset_stat(ds.handle, k) for k in ("fwd_segmented", "bwd_segmented", "fwd_single_launch", "bwd_single_launch", "hv_bytes")]
        grad, Hv, diag, ws = torch.empty_like(w), torch.empty_like(w), torch.empty_like(w), torch.zeros_like(w)
        out.append(ds.fun_grad(0, 0.5, w, grad))
        out.append(ds.hv(0.5, v, Hv))
        ds.hess_diag(0.5, diag)
        r = ds.solve(0, 0.5, 1e-3, ws)
        out += [r.f, r.cg_iters_total, grad.cpu().numpy().tobytes(), Hv.cpu().numpy().tobytes(), diag.cpu().numpy().tobytes(), ws.cpu().numpy().tobytes()]
        return out
    finally:
        ds.close()


SHAPES = {
    "one entry": lambda rng: (1, 1, [1], 0),
    "entries in one chunk": lambda rng: (40, 300, rng.integers(0, 30, 40), 0),
    "two chunks exactly": lambda rng: (128, 70, np.full(128, 32), 0),
    "empty rows first, between and last": lambda rng: (3000, 700, np.where((np.arange(3000) % 7 == 0) & (np.arange(3000) > 20) & (np.arange(3000) < 2900), 40, 0), 0),
    "one row of many chunks": lambda rng: (50, 9000, np.concatenate([rng.integers(0, 9, 20), [9000], rng.integers(0, 9, 29)]), 0),
    "columns of many chunks": lambda rng: (9000, 1200, rng.integers(0, 6, 9000), 4),
    "256 columns: one pass of the sort": lambda rng: (2000, 256, rng.integers(0, 60, 2000), 0),
    "257 columns: two": lambda rng: (2000, 257, rng.integers(0, 60, 2000), 0),
    "more than 65,536 columns: three": lambda rng: (3000, 70_001, rng.integers(0, 90, 3000), 3),
    "rows longer than a wavefront's share of the sort": lambda rng: (400, 3000, rng.integers(900, 2047, 400), 0),
}


def compare(rng, n, d, counts, popular, segmented):
    import paper_2008_03433_amd as tron
    arrays = csr(rng, n, d, counts, popular)
    tron.tron_tuning_set("csr_parts", 1)
    tron.tron_tuning_set("csr_segmented", segmented)
    tron.tron_tuning_set("csr_device_build", 0)
    want = results(n, d, arrays, False)
    tron.tron_tuning_set("csr_device_build", 1)
    assert results(n, d, arrays, False) == want
    assert results(n, d, arrays, True) == want


@pytest.mark.parametrize("segmented", [-1, 0, 1])
@pytest.mark.parametrize("name", SHAPES)
def test_the_same_layouts_as_on_the_host(rng, name, segmented):
    compare(rng, *SHAPES[name](rng), segmented)


def ends(n):
    counts = np.zeros(n, dtype=np.int64)
    counts[:20] = counts[-20:] = 20
    counts[n // 2] = 3
    return counts


# A chunk of entries between which there are so many empty rows or columns that its positions are looked up: 8 x 2048 rows are the last that are walked
EMPTY = {
    "16,384 rows of which the ends have entries": lambda rng: (16_384, 400, ends(16_384), 0),
    "16,385 rows of which the ends have entries": lambda rng: (16_385, 400, ends(16_385), 0),
    "a run of empty rows before a chunk that is full": lambda rng: (40_000, 400, ends(40_000) * 5, 0),
    "more empty columns than eight chunks": lambda rng: (300, 40_000, rng.integers(0, 6, 300), 3),
}


@pytest.mark.parametrize("segmented", [-1, 0, 1])
@pytest.mark.parametrize("name", EMPTY)
def test_the_same_layouts_with_long_runs_of_empty_rows(name, segmented):
    rng = np.random.default_rng(len(name))
    compare(rng, *EMPTY[name](rng), segmented)


@pytest.mark.parametrize("on_device", [False, True])
def test_the_same_errors_as_on_the_host(rng, on_device):
    import paper_2008_03433_amd as tron
    n, d = 500, 900
    rowptr, cols, val, y = csr(rng, n, d, rng.integers(1, 40, n))
    k = rowptr[:-1]

    def message(build, c, v):
        tron.tron_tuning_set("csr_device_build", build)
        with pytest.raises(tron.TronError) as e:
            arrays = (rowptr, c, v, y)
            tron.Dataset.from_csr(n, d, *([dev(a) for a in arrays] if on_device else arrays))
        return str(e.value)

    long = int(np.argmax(np.diff(rowptr)))
    faults = []
    for place, value in ((k[100], -1), (k[100], d), (k[long] + 1, int(cols[k[long]])), (k[long] + 2, int(cols[k[long]])), (k[0], -5), (rowptr[n] - 1, d + 7)):
        c = cols.copy()
        c[place] = value
        faults.append((c, val))
    for place, value in ((k[200], np.nan), (rowptr[n] - 1, np.inf), (0, -np.inf)):
        v = val.copy()
        v[place] = value
        faults.append((cols, v))
    c, v = cols.copy(), val.copy()   # two: the first in row order is told
    c[k[300]], v[k[299]] = d, np.nan
    faults.append((c, v))
    for c, v in faults:
        assert message(1, c, v) == message(0, c, v)
    tron.tron_tuning_set("csr_device_build", 1)
    tron.Dataset.from_csr(n, d, rowptr, cols, val, y).close()   # and goes on

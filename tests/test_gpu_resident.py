"""Solves in one launch, whose workgroups wait for each other inside the kernel, against the same solve with a launch per round."""
import ctypes
import threading
import time

import numpy as np
import pytest

import paper_2008_03433_amd as tron
from datagen import DenseProblem, SparseProblem
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


def _ways(ds):
    """Solves of the handle that ran as one launch, and those that gave that up."""
    return tuple(tron.tron_dataset_stat(ds.handle, name) for name in ("solves_in_one_launch", "solves_given_up"))


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
            before = np.array(_ways(ds))
            one = _solve(ds, loss, 0.3, start)
            assert _solve(ds, loss, 0.3, start) == one
            assert tuple(_ways(ds) - before) == (2, 0)
            knob("solve_wait_us", 0)    # every workgroup gives up at once, the solve starts again with a launch per round
            assert _solve(ds, loss, 0.3, start) == one
            assert tuple(_ways(ds) - before) == (2, 1)
            knob("solve_wait_us", -1)
            knob("solve_resident", 0)
            assert _solve(ds, loss, 0.3, start) == one
            assert tuple(_ways(ds) - before) == (2, 1)
            knob("solve_resident", 1)   # as where other solves hold the GPU
            assert _solve(ds, loss, 0.3, start) == one
            assert tuple(_ways(ds) - before) == (2, 1)
            knob("solve_resident", -1)
            assert _solve(ds, loss, 0.3, start) == one
            assert tuple(_ways(ds) - before) == (3, 1)
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
            out[k] = [_solve(ds, LOSS_L2SVM, 0.3, w0) for _ in range(5)], _ways(ds)[1]   # (some in one launch, some beside others: none given up)
            ds.close()

    for k in range(len(problems)):
        work(k, alone)
    threads = [threading.Thread(target=work, args=(k, together)) for k in range(len(problems))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert together == alone


def test_a_small_solve_does_not_wait_for_what_another_thread_s_stream_is_busy_with():
    """A solve that fills the GPU has its place from the call on, also while its launch waits behind other work of its stream (here one
    thread that sleeps).  A small solve of another thread goes on without one launch then, with the same bits."""
    torch = torch_mod()
    rng = np.random.default_rng(13)
    w0 = torch.zeros(24, dtype=torch.float64, device="cuda")
    busy = torch.cuda.Stream()
    with torch.cuda.stream(busy):
        large = tron.Dataset.from_problem(_dense(rng, 120_000, 24))
    small = tron.Dataset.from_problem(_dense(rng, 20_000, 24))
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    try:
        one = _solve(small, LOSS_LR, 0.3, w0)
        with torch.cuda.stream(busy):
            other = _solve(large, LOSS_LR, 0.3, w0)
            torch.cuda._sleep(1000)   # its first launch takes longer
            ends[0].record()
            torch.cuda._sleep(10_000_000)
            ends[1].record()
        torch.cuda.synchronize()
        per_second = 1e10 / ends[0].elapsed_time(ends[1])
        results = []
        w = w0.clone()
        torch.cuda.synchronize()
        with torch.cuda.stream(busy):
            torch.cuda._sleep(int(0.5 * per_second))
            ends[1].record()
        thread = threading.Thread(target=lambda: results.append(large.solve(LOSS_LR, 0.3, 1e-4, w)))
        thread.start()
        time.sleep(0.1)   # the thread is in its solve
        assert _solve(small, LOSS_LR, 0.3, w0) == one
        asleep = not ends[1].query()
        thread.join()
        assert asleep
        assert ends[1].query() and results[0].f == other[1] and w.cpu().numpy().tobytes() == other[0]
        assert _ways(small) == (1, 0) and _ways(large) == (2, 0)
    finally:
        torch.cuda.synchronize()
        large.close()
        small.close()


# one counter (up to 64 workgroups of 512 rows) and eight groups with one each
@pytest.mark.parametrize("n", [20_000, 120_000])
def test_a_launch_behind_one_that_was_given_up_finds_the_counters_at_zero(knob, n):
    torch = torch_mod()
    ds = tron.Dataset.from_problem(_dense(np.random.default_rng(n), n, 24))
    w0 = torch.zeros(24, dtype=torch.float64, device="cuda")
    try:
        one = _solve(ds, LOSS_L2SVM, 0.3, w0)
        for _ in range(40):
            knob("solve_wait_us", 0)
            assert _solve(ds, LOSS_L2SVM, 0.3, w0) == one
            knob("solve_wait_us", -1)
            assert _solve(ds, LOSS_L2SVM, 0.3, w0) == one
        assert _ways(ds) == (41, 40)
    finally:
        ds.close()


def test_solve_on_a_stream_that_may_use_a_quarter_of_the_compute_units():
    """Workgroups for all of them could not be resident together there: such a solve takes a launch per round and waits for nothing."""
    torch = torch_mod()
    hip = tron.load_library()   # its own symbols and those of the runtime that it is linked against
    w0 = torch.zeros(24, dtype=torch.float64, device="cuda")
    stream, words = ctypes.c_void_p(), torch.cuda.get_device_properties(0).multi_processor_count // 32
    mask = (ctypes.c_uint32 * words)(*([0xFFFFFFFF] * (words // 4) + [0] * (words - words // 4)))
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), words, mask) == 0
    rng = np.random.default_rng(7)
    for n, here in ((20_000, True), (120_000, False)):   # 40 workgroups, 235
        p = _dense(rng, n, 24)
        results = []
        for masked in (True, False):
            with torch.cuda.stream(torch.cuda.ExternalStream(stream.value) if masked else torch.cuda.Stream()):
                ds = tron.Dataset.from_problem(p)
                results.append([_solve(ds, LOSS_LR, 0.3, w0) for _ in range(3)])
                assert _ways(ds) == ((3, 0) if here or not masked else (0, 0))
                ds.close()
        assert results[0] == results[1]
    torch.cuda.synchronize()
    assert hip.hipStreamDestroy(stream) == 0


@pytest.mark.parametrize("sparse", [False, True])
def test_solves_that_were_given_up_are_not_tried_again_at_once(knob, sparse):
    """What held a part of the GPU may hold it for long: one wait, then one solve the other way, another wait, two solves, four, ..."""
    torch = torch_mod()
    rng = np.random.default_rng(5)
    ds = tron.Dataset.from_problem(_sparse(rng, 500, 400, 9) if sparse else _dense(rng, 5000, 24))
    w0 = torch.zeros(400 if sparse else 24, dtype=torch.float64, device="cuda")
    try:
        one = _solve(ds, LOSS_LR, 0.3, w0)
        assert _ways(ds) == (1, 0)
        knob("solve_wait_us", 0)
        given_up = []
        for _ in range(20):
            other = _solve(ds, LOSS_LR, 0.3, w0)
            assert other[3:6] == one[3:6] and abs(other[1] - one[1]) <= 1e-12 * abs(one[1])
            given_up.append(_ways(ds)[1])
        assert given_up == [1, 1, 2, 2, 2] + [3] * 5 + [4] * 9 + [5]
        knob("solve_wait_us", -1)   # another limit: afresh
        assert _solve(ds, LOSS_LR, 0.3, w0) == one and _ways(ds) == (2, 5)
        knob("solve_wait_us", 0)
        _solve(ds, LOSS_LR, 0.3, w0)
        assert _ways(ds) == (2, 6)
        knob("solve_resident", 0)   # not to be tried anyway: no solve counts
        for _ in range(3):
            _solve(ds, LOSS_LR, 0.3, w0)
        knob("solve_resident", -1)
        _solve(ds, LOSS_LR, 0.3, w0)
        _solve(ds, LOSS_LR, 0.3, w0)
        assert _ways(ds) == (2, 7)
    finally:
        ds.close()


# ------------------------------------------------------------------ sparse
def _sparse(rng, n, d, mean, common=(), long_rows=(), zipf=0.0):
    """Rows of about `mean` entries; columns `common` are in every row, the rows `long_rows` have two thirds of all columns, every
    seventh row and the columns after 0.9 d are empty (but for those)."""
    p = np.arange(1, d + 1, dtype=np.float64) ** -zipf
    p[int(0.9 * d) + 1:] = 0.0
    p = np.cumsum(p / p.sum())
    rows, cols = [], []
    for i in range(n):
        k = 0 if i % 7 == 6 else rng.poisson(mean)
        c = np.minimum(np.searchsorted(p, rng.random(k)), d - 1)
        if i in long_rows:
            c = rng.permutation(d)[:2 * d // 3]
        c = np.unique(np.concatenate([c, np.asarray(common, dtype=c.dtype)])).astype(np.int32)
        rows.append(c.size)
        cols.append(c)
    rowptr = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    col = np.concatenate(cols) if cols else np.zeros(0, np.int32)
    val = rng.lognormal(size=col.size) / np.sqrt(np.repeat(np.maximum(rows, 1), rows))
    score = np.zeros(n)
    np.add.at(score, np.repeat(np.arange(n), rows), val * rng.standard_normal(d)[col])
    y = np.where(score + 0.3 * rng.standard_normal(n) >= 0.0, 1.0, -1.0)
    return SparseProblem("resident", n, d, rowptr, col, val, y)


# one entry; fewer entries than a chunk of 2048; rows and columns of several lengths with many short ones in a chunk; columns
# longer than a chunk (the transposed copy as segments) and rows longer than a chunk (the other one); more chunks than the
# workgroups hold at once (512); more rows in a chunk than the launch takes (the other path, in both cases)
SPARSE = {
    "one": dict(n=1, d=1, mean=0, common=(0,)),
    "tiny": dict(n=9, d=13, mean=3),
    "chunk": dict(n=60, d=41, mean=30),
    "short": dict(n=2500, d=2000, mean=4),
    "columns": dict(n=6000, d=3000, mean=12, common=(5, 1700), zipf=1.05),
    "rows": dict(n=300, d=9000, mean=60, long_rows=(0, 17, 18, 299)),
    "both": dict(n=5000, d=5000, mean=10, common=(0, 2600), long_rows=(3, 4000)),
    "rounds": dict(n=30_000, d=20_000, mean=55, zipf=0.8),
    "wide": dict(n=400, d=60_000, mean=12),
}


def _same_solve(a, b, rel):
    """The same trajectory, the numbers within rel.  (Rounding of 1e-16 per sum, which the inner iterations amplify: up to 5e-9 in w
    over forty problems of this kind.)"""
    wa, wb = np.frombuffer(a[0]), np.frombuffer(b[0])
    assert np.linalg.norm(wa - wb) <= rel * max(np.linalg.norm(wb), 1e-300)
    assert abs(a[1] - b[1]) <= rel * abs(b[1])
    assert (a[3], a[4], a[5]) == (b[3], b[4], b[5])
    for s, t in zip(a[6], b[6]):
        assert [s[k] for k in ("iter", "cg_iters", "accepted", "on_boundary")] == [t[k] for k in ("iter", "cg_iters", "accepted", "on_boundary")]
        assert abs(s["f"] - t["f"]) <= rel * abs(t["f"]) and abs(s["delta"] - t["delta"]) <= 1e3 * rel * abs(t["delta"])


@pytest.mark.parametrize("loss", [LOSS_LR, LOSS_L2SVM])
@pytest.mark.parametrize("name", SPARSE)
def test_sparse_solve_in_one_launch_follows_the_solve_driven_by_the_host(rng, knob, loss, name):
    _follows_the_host(rng, knob, loss, _sparse(rng, **SPARSE[name]), None)


# Shapes that must take the one launch, whatever ran before (their inputs are their own): both orientations plain, one or both as segments
# (forced, where a chunk of long rows alone would stay plain), two and three rounds of chunks (more than 512 and 1024 of them).  The
# shapes above take it or leave it, as their rows fall: "rounds" and "wide" have too many empty columns in a chunk.
ONE_LAUNCH = {
    "tiny": dict(n=9, d=13, mean=3), "plain": dict(n=3000, d=2500, mean=9), "columns": dict(n=6000, d=3000, mean=12, common=(5, 1700), zipf=1.05),
    "rows": dict(n=300, d=9000, mean=60, long_rows=(0, 17, 18, 299)), "both": dict(n=5000, d=5000, mean=10, common=(0, 2600), long_rows=(3, 4000)),
    "two rounds": dict(n=30_000, d=12_000, mean=50), "three rounds": dict(n=60_000, d=16_000, mean=50, long_rows=(3, 40_000)),
}


@pytest.mark.parametrize("loss", [LOSS_LR, LOSS_L2SVM])
@pytest.mark.parametrize("name", ONE_LAUNCH)
def test_sparse_solve_takes_the_one_launch(knob, loss, name):
    rng = np.random.default_rng(len(name))
    if name in ("rows", "three rounds"):
        knob("csr_segmented", 1)
    _follows_the_host(rng, knob, loss, _sparse(rng, **ONE_LAUNCH[name]), True)


def _follows_the_host(rng, knob, loss, q, one_launch):
    """one_launch: whether the solves are known to take it (None: either way)."""
    torch = torch_mod()
    ds = tron.Dataset.from_problem(q)
    zero = torch.zeros(q.d, dtype=torch.float64, device="cuda")
    far = torch.from_numpy(3.0 * rng.standard_normal(q.d)).cuda()
    try:
        # C so small, and from far away the inner solves so short, that rounding stays small: with C = 1 the L2-SVM solve of "columns"
        # takes 78 products, and the host-driven solve itself moves by 5e-2 in w when its start moves by one part in 1e15.
        # Not preconditioned by the whole diagonal: of one column that is the Hessian, and the step then ends exactly at the radius.
        far_kw = dict(max_cg=12, max_outer=4)
        for start, C, kw in ((zero, 0.02, {}), (far, 0.02, far_kw), (zero, 0.02, dict(precond_blend=0.3)), (far, 0.02, dict(precond_blend=0.9, **far_kw)),
                             (zero, 0.02, dict(max_outer=1)), (zero, 0.02, dict(max_cg=2, trace_cap=1))):
            def solve():
                w = start.clone()
                r = ds.solve(loss, C, 0.01, w, **kw)
                hv = torch.empty_like(w)
                ds.hv(C, far, hv)   # with the D that the solve leaves
                return w.cpu().numpy().tobytes(), r.f, r.gnorm, r.outer_iters, r.cg_iters_total, r.status, r.trace, hv.cpu().numpy()

            before = np.array(_ways(ds))
            one = solve()
            here = tron.tron_dataset_stat(ds.handle, "solves_in_one_launch") - before[0]
            assert here == 1 or not one_launch
            if here:   # a launch per step, as where other solves hold the GPU: the same rows and sums in the same order
                knob("solve_resident", 1)
                assert solve()[:7] == one[:7] and solve()[:7] == one[:7]
                knob("solve_resident", -1)
                assert tuple(_ways(ds) - before) == (1, 0)
            again = solve()
            assert one[:7] == again[:7]
            knob("solve_wait_us", 0)    # every workgroup gives up at once, the host drives the solve
            given_up = solve()
            knob("solve_wait_us", -1)
            assert tuple(_ways(ds) - before) == (2 * here, here)
            assert solve()[:7] == one[:7]
            knob("solve_resident", 0)
            host = solve()
            knob("solve_resident", -1)
            assert tuple(_ways(ds) - before) == (3 * here, here)
            assert given_up[:7] == host[:7]
            _same_solve(one, host, 5e-9)
            assert np.linalg.norm(one[7] - host[7]) <= 1e-7 * np.linalg.norm(host[7])
    finally:
        ds.close()


def test_sparse_solve_of_many_steps_goes_on_in_further_launches(rng, knob):
    """More than 512 products, the most of one launch, and more records than the pinned ones (32)."""
    torch = torch_mod()
    q = _sparse(rng, 1500, 400, 20, common=(3,))
    ds = tron.Dataset.from_problem(q)
    w0 = torch.zeros(q.d, dtype=torch.float64, device="cuda")
    try:
        for kw in (dict(cg_xi=1e-9), dict(max_cg=2, max_outer=60)):
            def solve():
                w = w0.clone()
                return ds.solve(LOSS_LR, 1e3, 1e-7, w, **kw), w

            one, w = solve()
            assert _ways(ds) == (1 if "cg_xi" in kw else 2, 0)
            knob("solve_resident", 0)
            host, v = solve()
            knob("solve_resident", 1)
            steps, v1 = solve()
            knob("solve_resident", -1)
            assert steps == one and torch.equal(v1, w)
            if "cg_xi" in kw:   # the same minimiser: the gradient is 1e-7 of the first one, H >= I
                assert one.n_hv > 256 and one.status == host.status == 0
                assert abs(one.f - host.f) <= 1e-9 * host.f
            else:
                assert one.outer_iters == host.outer_iters > 32 and len(one.trace) == len(host.trace)
                assert [t["iter"] for t in one.trace] == list(range(1, one.outer_iters + 1))
                assert abs(one.f - host.f) <= 1e-6 * host.f
    finally:
        ds.close()


@pytest.mark.parametrize("name", ["columns", "two rounds", "three rounds"])
def test_sparse_solves_whose_wait_is_short_have_the_bits_of_one_launch(knob, name):
    """A limit of a microsecond, which some of the waits exceed and some do not: whether a solve is given up in the middle, is not tried or
    ends as one launch, its bits are the same."""
    torch = torch_mod()
    q = _sparse(np.random.default_rng(3), **ONE_LAUNCH[name])
    if name == "three rounds":
        knob("csr_segmented", 1)
    ds = tron.Dataset.from_problem(q)
    w0 = torch.zeros(q.d, dtype=torch.float64, device="cuda")
    try:
        one = _solve(ds, LOSS_LR, 0.3, w0)
        for _ in range(3):
            knob("solve_wait_us", 1)
            for _ in range(6):
                assert _solve(ds, LOSS_LR, 0.3, w0) == one
            knob("solve_wait_us", -1)
            assert _solve(ds, LOSS_LR, 0.3, w0) == one
    finally:
        ds.close()


def _solve_with_records(ds, w0, many, records):
    """A solve that may leave `many` records, few of which it will, in an array of fewer."""
    from paper_2008_03433_amd import binding
    w, res = w0.clone(), binding._Result()
    res.trace_cap, res.trace = many, ctypes.addressof(records)
    params = binding._Params(LOSS_LR, 0.3, 1e-4, many, 1000, 0.1, 0.0)
    status = tron.load_library().tron_solve(ds.handle, ctypes.byref(params), w.data_ptr(), ctypes.byref(res))
    trace = [{name: getattr(records[k], name) for name, _ in binding.TraceRec._fields_} for k in range(res.trace_len)]
    return w.cpu().numpy().tobytes(), res.f, res.gnorm, res.outer_iters, res.cg_iters_total, status, trace


def test_sparse_solve_with_room_for_any_number_of_records(knob):
    """Up to a million records the work space holds them; for more the host drives the solve, and takes no memory for them."""
    torch = torch_mod()
    from paper_2008_03433_amd import binding
    q = _sparse(np.random.default_rng(17), **ONE_LAUNCH["plain"])
    ds = tron.Dataset.from_problem(q)
    w0, records = torch.zeros(q.d, dtype=torch.float64, device="cuda"), (binding.TraceRec * 1000)()
    try:
        one = _solve(ds, LOSS_LR, 0.3, w0)
        assert _solve_with_records(ds, w0, 2**20, records) == one and _ways(ds) == (2, 0)
        knob("solve_resident", 0)
        host = _solve(ds, LOSS_LR, 0.3, w0)
        knob("solve_resident", -1)
        free = torch.cuda.mem_get_info()[0]
        for many in (2**20 + 1, 2**31 - 1):
            assert _solve_with_records(ds, w0, many, records) == host and _ways(ds) == (2, 0)
        assert torch.cuda.mem_get_info()[0] >= free - 2**27
        assert _solve(ds, LOSS_LR, 0.3, w0) == one and _ways(ds) == (3, 0)
    finally:
        ds.close()


@pytest.mark.parametrize("shapes", [("two rounds", "columns", "both", "plain"), ("two rounds", "three rounds", "two rounds")])
def test_sparse_solves_of_threads_that_fill_the_gpu_have_the_bits_they_have_alone(shapes):
    """Several grids of all compute units, and one of them among small ones."""
    rng = np.random.default_rng(11)
    _threads([_sparse(rng, **ONE_LAUNCH[k]) for k in shapes], (1, 3))


def test_sparse_solves_of_several_threads_on_streams_of_their_own(rng):
    _threads([_sparse(rng, **SPARSE[k]) for k in ("columns", "rounds", "both", "short")], (5,))


def _threads(problems, solves):
    torch = torch_mod()
    alone, together = {}, {}

    def work(k, out):
        with torch.cuda.stream(torch.cuda.Stream()):
            ds = tron.Dataset.from_problem(problems[k])
            w0 = torch.zeros(problems[k].d, dtype=torch.float64, device="cuda")
            out[k] = [_solve(ds, LOSS_LR, 0.3, w0) for _ in range(sum(solves))], _ways(ds)[1]   # (some in one launch, some beside others: none given up)
            ds.close()

    for k in range(len(problems)):
        work(k, alone)
    threads = [threading.Thread(target=work, args=(k, together)) for k in range(len(problems))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert together == alone

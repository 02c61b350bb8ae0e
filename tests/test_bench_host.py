"""Host logic of bench.py that needs no GPU: the committed rocprofv3 summaries are read back as bytes per launch."""
import importlib.util
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench():
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _format_bytes(b, workload, slot):
    """The bytes in the stored format that the summary was taken with."""
    kname, fname = b.ROCPROF_NAMES[(workload, slot)]
    columns = None
    for line in open(os.path.join(ROOT, "profiles", fname)):
        cells = [c.strip() for c in line.strip().strip("|").split("|")]
        if cells[0] == "kernel":
            columns = cells
        if cells[0] == f"`{kname}`" and "format GB" in columns:
            return float(cells[columns.index("format GB")]) * 1e9
    raise AssertionError((workload, slot, kname))


def test_traffic_is_read_from_the_committed_summaries_in_bytes():
    b = _bench()
    # what the kernels of each profiled workload move per launch lies between a few MB and a few tens of GB, and
    # within a factor of two of known sizes: c5 is 44.2 GB of matrix, the hot rows of c3 without values read 0.36 GB
    seen = {}
    for (workload, slot) in b.ROCPROF_NAMES:
        stored = _format_bytes(b, workload, slot)
        t = b.measured_traffic(workload, slot, stored)
        assert t is not None and 1e6 < t < 1e11 and 0.95 < t / stored < 1.2, (workload, slot, t)
        seen[(workload, slot)] = t
        # a kernel that has other bytes to move is not the one that was measured
        assert b.measured_traffic(workload, slot, 0.97 * stored) is None and b.measured_traffic(workload, slot, 1.03 * stored) is None
    assert 0.9 < seen[("c5", "dense_hv")] / (8.0 * 230_000_000 * 24) < 1.1
    assert 0.3e9 < seen[("c3", "spmv_tiles")] < 0.6e9
    assert seen[("c3_values", "spmv_tiles")] > 2.0 * seen[("c3", "spmv_tiles")]   # the value stream triples the bytes
    assert b.measured_traffic(None, "spmv_tiles", 1e9) is None and b.measured_traffic("c3", "no_such_kernel", 1e9) is None


def test_the_measured_kernels_are_in_the_library():
    import paper_2008_03433_amd as tron
    b = _bench()
    lib = open(tron.lib_path(), "rb").read()
    for kname, _ in b.ROCPROF_NAMES.values():
        name, _, args = kname.partition("<")
        mangled = f"{len(name)}{name}"
        if args:
            mangled += "I" + "".join({"true": "Lb1E", "false": "Lb0E"}.get(a, f"Li{a}E") for a in args.rstrip(">").split(", ")) + "E"
        assert mangled.encode() in lib, kname


def test_the_pass_kernel_named_is_the_one_of_the_library_s_rule():
    b = _bench()
    matrix, vector = "fp64 matrix instructions", "vector units"
    assert [b.pass_kernel(1_000_000, 24, K, "lr") for K in (6, 8, 9)] == [vector, vector, matrix]
    assert [b.pass_kernel(20_000_000, 24, K, "lr") for K in (7, 8, 12)] == [vector, matrix, matrix]
    assert [b.pass_kernel(1000, d, 7, "lr") for d in (25, 26, 27, 28, 32)] == [vector, matrix, vector, matrix, matrix]
    assert [b.pass_kernel(20_000_000, 32, K, "l2svm") for K in (6, 8, 9)] == [vector, vector, matrix]
    src = open(os.path.join(ROOT, "paper_2008_03433_amd", "csrc", "batch.hip")).read()
    assert "mfma_from[2] = {s.L == 4 && s.E == 8 ? 7 : read_once(n, d) ? 8 : 9, 9};" in src   # what is said above


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in (r.stdout + r.stderr)


def test_the_line_on_stdout_is_short_whatever_the_record_holds():
    b = _bench()
    x = 1234567.890123456
    roofline = {"kernel": "spmv_tiles", "in": "kernels_hv", "bound": "hbm", "achieved": x, "peak": 8000.0, "unit": "GB/s", "frac": x, "traffic": x,
                "ms_per_launch": x, "format_bytes_per_launch": x, "work_GB/s": x, "workload": "w" * 40, "note": "n" * 400, "also": [{"kernel": "k"}] * 30}
    call = {"per_s": x, "ms": x, "GB/s": x, "frac_hbm_peak": x}
    out = {"metric": "m" * 107, "value": x, "unit": "Hv/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": x, "higher_is_better": True,
           "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic", "config": {f"key{i}": x for i in range(12)},
           "solve": {"outer_iters": 5, "cg_iters": 22, "f": x, "converged": True, "min_seconds": x, "gnorm": x}, "hv_call": call, "roofline": roofline,
           "cpu_baseline": {"value": x, "unit": "Hv/s", "cores": 1, "kind": "oracle", "sample": "s" * 250, "host_cpu": "c" * 50},
           "also": {"c5": {"ms_per_step": x, "hv_call": call, "roofline": roofline}}, "others": {"c1": [x] * 1000}}
    line = b.headline(out)
    assert len(json.dumps(line)) < 2000
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config"):
        assert line[key] == b.short(out[key]), key
    assert line["roofline"]["kernel"] == "spmv_tiles" and "also" not in line["roofline"]
    assert abs(line["value"] / x - 1) < 1e-5
    out["cpu_baseline"] = None
    assert "cpu_baseline" not in b.headline(out)

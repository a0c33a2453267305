"""Host-side logic of bench.py, on the CPU: the one-GPU refusal, the dispatch keys that
join a plan with rocprofv3's kernel names (the measured-traffic lookup depends on
them), and the scaling of HBM counters by a plain copy."""
import csv
import json
import os
import subprocess
import sys

import pytest

import bench
import paper_2509_18344_amd as ss

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2 and "one GPU" in r.stderr, (r.returncode, r.stderr)


# Kernels, grids and workgroups (work-items) that rocprofv3 recorded for launches of
# bench.py's workloads on an MI355X (profiles/qlinear_suite_kernel_trace.md); of those whose
# plan follows from the shape alone (others ask the GPU how many workgroups fit).
TRACED = [
    ((1, 7168, 5120, 3, 128), "subspec::(anonymous namespace)::k_qstream<3, 128, 2, 16, 2, 1>", 229376, 1024),
    ((1, 3584, 18944, 4, 128), "subspec::(anonymous namespace)::k_qstream<4, 128, 1, 16, 4, 1>", 229376, 1024),
    ((1, 512, 256, 4, 64), "subspec::(anonymous namespace)::k_qstream<4, 64, 1, 4, 3, 1>", 8192, 256),
    ((1, 55296, 5120, 3, 128), "subspec::k_qgemv<3, 128, 1, 1, 2, 4, 2>", 245760, 256),
    ((16, 7168, 5120, 3, 128), "subspec::k_qgemm_mfma<3, 128, 1, 1, 2, 4, 2>", 114688, 256),
    ((64, 5120, 5120, 3, 128), "subspec::qmma::k_qmma<3, 128, 1, 1, 4, 8, 2>", 122880, 512),
    ((128, 5120, 5120, 3, 128), "subspec::qmma::k_qmma<3, 128, 1, 1, 4, 8, 2>", 81920, 512),
    ((128, 7168, 5120, 3, 128), "subspec::qmma::k_qmma<3, 128, 1, 1, 4, 8, 2>", 114688, 512),
    ((64, 55296, 5120, 3, 128), "subspec::qmma::k_qmma<3, 128, 2, 1, 4, 8, 1>", 110592, 512),
    ((128, 55296, 5120, 2, 64), "subspec::qmma::k_qmma<2, 64, 4, 1, 4, 8, 1>", 110592, 512),
    ((48, 37888, 3584, 4, 128), "subspec::qmma::k_qmma<4, 128, 2, 1, 4, 8, 1>", 75776, 512),
]


@pytest.mark.parametrize("shape,name,grid_items,wg", TRACED)
def test_plan_key_matches_the_traced_kernel(shape, name, grid_items, wg):
    """A launch's key from its plan equals the key of the kernel and the whole grid (both
    dimensions) that a trace recorded for it, so the plan is what runs and its measured
    traffic is found."""
    key = bench.library_key(f"void {name}(subspec::QArgs)", grid_items, wg)
    with open(os.path.join(ROOT, "profiles", "qlinear_suite_kernel_trace.md"), encoding="utf-8") as f:
        assert f"`{key}`" in f.read()
    assert bench.plan_key(ss.subspec_qlinear_plan(*shape), *shape[3:]) == key


def test_library_key_ignores_other_kernels():
    assert bench.library_key("void at::native::vectorized_elementwise_kernel<4>(int)", 1024, 256) is None


def _counter_csv(d, rows):
    os.makedirs(d, exist_ok=True)
    with open(os.path.join(d, "run_counter_collection.csv"), "w", newline="") as f:
        w = csv.DictWriter(f, fieldnames=["Dispatch_Id", "Kernel_Name", "Grid_Size", "Workgroup_Size",
                                          "Counter_Name", "Counter_Value"])
        w.writeheader()
        for r in rows:
            w.writerow(r)


def test_counters_are_scaled_by_the_copy(tmp_path, monkeypatch):
    """FETCH_SIZE and WRITE_SIZE (KiB per dispatch, summed over the counter's
    instances) become bytes with the factors a copy of known size gives."""
    out = tmp_path / "traffic.json"
    fam = dict(bench.FAMILIES["qlinear"], json=str(out))
    monkeypatch.setitem(bench.FAMILIES, "qlinear", fam)
    name = "void subspec::qmma::k_qmma<3, 128, 4, 1, 4, 8, 1>(subspec::QArgs)"
    grid, wg = 110592, 512
    # two dispatches of one kernel, each counter reported by two instances
    fetch = [dict(Dispatch_Id=d, Kernel_Name=name, Grid_Size=grid, Workgroup_Size=wg, Counter_Name="FETCH_SIZE",
                  Counter_Value=v) for d, v in ((1, 30000.0), (1, 40000.0), (2, 35000.0), (2, 35000.0))]
    write = [dict(Dispatch_Id=d, Kernel_Name=name, Grid_Size=grid, Workgroup_Size=wg, Counter_Name="WRITE_SIZE",
                  Counter_Value=v) for d, v in ((1, 100.0), (1, 200.0), (2, 300.0), (2, 0.0))]
    copy = "void at::native::copy_kernel(int)"
    cfetch = [dict(Dispatch_Id=1, Kernel_Name=copy, Grid_Size=4096, Workgroup_Size=256, Counter_Name="FETCH_SIZE",
                   Counter_Value=512.0)]
    cwrite = [dict(Dispatch_Id=1, Kernel_Name=copy, Grid_Size=4096, Workgroup_Size=256, Counter_Name="WRITE_SIZE",
                   Counter_Value=1024.0)]
    for d, rows in (("f", fetch), ("w", write), ("cf", cfetch), ("cw", cwrite)):
        _counter_csv(tmp_path / d, rows)
    bench.summarize_pmc(str(tmp_path / "f"), str(tmp_path / "w"), str(tmp_path / "cf"), str(tmp_path / "cw"),
                        calib_bytes=1 << 20)
    res = json.loads(out.read_text())
    assert res["calibration"]["fetch_scale"] == 2.0 and res["calibration"]["write_scale"] == 1.0
    key = bench.library_key(name, grid, wg)
    e = res["kernels"][key]
    assert e["dispatches"] == 2 and e["fetch_kib_raw"] == 70000.0 and e["write_kib_raw"] == 300.0
    assert e["hbm_bytes_per_launch"] == int(round(70000.0 * 1024 * 2 + 300.0 * 1024))
    assert res["kernel_source_sha256_16"] == bench.kernel_source_hash("qlinear")

"""Names that bench.py gives the gather kernel's instantiations in a trace (the
destination kind stands before the chunks a workgroup takes), and the counters
of instantiations that share a name."""
import json

import pytest

import bench

ARGS = "(symten::CopyTask const*, long const*, int, long, symten::%s)"


@pytest.mark.parametrize("chunks", [1, 4])
@pytest.mark.parametrize("ptrs", ["ArgPtrs", "DevPtrs"])
@pytest.mark.parametrize("src,kind,name", [("float", 0, "f32,f32"), ("float", 2, "f32,bf16"), ("float", 3, "f32,bf16x2"),
                                           ("float", 4, "f32,acc"), ("float", 5, "f32,bf16x3"), ("double", 0, "f64,f32"),
                                           ("double", 1, "f64,f64"), ("double", 4, "f64,acc")])
def test_gather_names(src, kind, name, ptrs, chunks):
    traced = "void symten::copy_kernel<symten::%s, %s, %d, %d>" % (ptrs, src, kind, chunks) + ARGS % ptrs
    assert bench.profile_name(traced) == "copy_kernel<%s>" % name


def test_traffic_of_instantiations_that_share_a_name(tmp_path):
    copy = lambda chunks: "void symten::copy_kernel<symten::ArgPtrs, float, 0, %d>" % chunks + ARGS % "ArgPtrs"
    for c in ("FETCH_SIZE", "WRITE_SIZE"):
        rows = [{"kernel": copy(1), "counter": c, "dispatches": 30, "avg_per_dispatch": 10.0},
                {"kernel": copy(4), "counter": c, "dispatches": 10, "avg_per_dispatch": 50.0}]
        (tmp_path / ("pmc_%s.summary.json" % c)).write_text(json.dumps(rows))
        (tmp_path / ("pmc_copy_%s.summary.json" % c)).write_text(json.dumps(
            [{"kernel": "__amd_rocclr_copyBuffer", "counter": c, "dispatches": 5, "avg_per_dispatch": 262144.0}]))
    k = bench.write_traffic(str(tmp_path), "w", "cmd", out=str(tmp_path / "t.json"))["kernels"]["copy_kernel<f32,f32>"]
    assert k["fetch_size_dispatches"] == k["write_size_dispatches"] == 40
    assert k["fetch_size_kib_per_dispatch"] == pytest.approx(20.0)
    assert k["bytes_per_launch"] == pytest.approx(2 * 20 * 1024)

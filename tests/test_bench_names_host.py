"""Names that bench.py gives the gather kernel's instantiations in a trace: the
destination kind stands before the chunks a workgroup takes."""
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

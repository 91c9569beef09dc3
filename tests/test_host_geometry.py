"""The library's host-side launch geometry (csrc/geometry.h), compiled with g++ and checked without a GPU."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def geo(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("geometry") / "geometry_shim.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2607_06202_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host", "geometry_shim.cpp"), "-o", so])
    return ctypes.CDLL(so)


def plan(geo, R, E, k, Tr, H, count_groups=0, sync=0, capacity=1280, cus=256):
    out = (ctypes.c_int * 6)()
    geo.plan_decomposed(R, E, k, Tr, H, count_groups, sync, capacity, cus, out)
    return dict(zip(("grid", "count_groups", "send_groups", "senders", "batch", "combine_run"), out))


@pytest.mark.parametrize("sync", [0, 1, 2, 3])
@pytest.mark.parametrize("k", [1, 8])
@pytest.mark.parametrize("count_groups", [1280, 1 << 30, (1 << 31) - 1 - 1280, (1 << 31) - 2, (1 << 31) - 1])
def test_count_groups_beyond_the_device_give_a_grid_beyond_it(geo, sync, k, count_groups):
    """A launch whose workgroups wait for each other must not start unless all of them fit on the device at
    once: the caller compares grid with capacity, so the grid's sum must not wrap below it."""
    p = plan(geo, 64, 256, k, 128, 7168, count_groups, sync)
    assert p["count_groups"] == count_groups and p["grid"] > 1280


@pytest.mark.parametrize("T,pieces", [
    (8 * 4194304, 2),              # 32M tokens of 520 columns: 2^32 threads at two waves per workgroup
    (4793491, 14),                 # 64 GiB of 7168-column tokens
    ((1 << 31) - 2, 1), ((1 << 31) - 2, 2048),
    (1, 1), (3, 1), (8192, 14)])
@pytest.mark.parametrize("per_group,threads", [(2, 128), (4, 256)])
def test_row_kernel_grids_stay_below_the_launch_limit(geo, T, pieces, per_group, threads):
    """gridDim * blockDim < 2^32, every unit within a strided grid's reach, and one workgroup per
    per_group units wherever that many fit."""
    geo.unit_grid.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    geo.unit_grid.restype = ctypes.c_uint
    n = geo.unit_grid(T * pieces, per_group, threads)
    want = -(-T * pieces // per_group)
    assert 1 <= n and n * threads < 1 << 32
    assert n == want or (n < want and (n + 1) * threads >= 1 << 32)

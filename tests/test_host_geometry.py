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


GENERAL, FEW, WIDE, SPLIT = range(4)  # the forms of the one-launch kernel


def plan(geo, R, E, k, Tr, H, count_groups=0, sync=0, form=None, capacity=1280, cus=256):
    out = (ctypes.c_int * 6)()
    if form is None:
        form = geo.decomposed_form(R, E, k, Tr, H, sync)
    geo.plan_decomposed(R, E, k, Tr, H, count_groups, sync, form, capacity, cus, out)
    return dict(zip(("grid", "count_groups", "send_groups", "senders", "batch", "combine_run"), out), form=form)


@pytest.mark.parametrize("sync", [0, 1, 2, 3])
@pytest.mark.parametrize("k", [1, 8])
@pytest.mark.parametrize("count_groups", [1280, 1 << 30, (1 << 31) - 1 - 1280, (1 << 31) - 2, (1 << 31) - 1])
def test_count_groups_beyond_the_device_give_a_grid_beyond_it(geo, sync, k, count_groups):
    """A launch whose workgroups wait for each other must not start unless all of them fit on the device at
    once: the caller compares grid with capacity, so the grid's sum must not wrap below it."""
    for form in (None, SPLIT) if sync else (None,):
        p = plan(geo, 64, 256, k, 128, 7168, count_groups, sync, form)
        assert p["count_groups"] == count_groups and p["grid"] > 1280


@pytest.mark.parametrize("sync", [0, 1, 2, 3])
def test_one_launch_plans(geo, sync):
    """Every plan over a grid of shapes and splits: all workgroups fit on the device, a batch has a wave for
    each token's placement, every send workgroup has a batch (one without would go on to combine without having
    waited for the offsets), no combine task is empty, and the split form keeps a workgroup that combines."""
    forms = set()
    for R in (1, 4, 32, 64, 256):
        for k in (1, 2, 3, 8, 32):
            for Tr in (1, 2, 5, 16, 128, 300, 1024):
                for H in (8, 256, 512, 520, 2048, 4992, 7168, 1 << 20):
                    for count_groups, capacity in ((0, 1280), (0, 1792), (1, 1280), (7, 1536), (1000, 1280), (1278, 1280)):
                        p = plan(geo, R, R * (256 // R), k, Tr, H, count_groups, sync, capacity=capacity)
                        what = (R, k, Tr, H, count_groups, p)
                        T, chunks = R * Tr, -(-H // 512)
                        assert p["grid"] <= capacity and 1 <= p["batch"] <= 4, what
                        assert 1 <= p["send_groups"] <= -(-T // p["batch"]), what
                        assert 1 <= p["combine_run"] <= chunks, what
                        n = p["count_groups"] + p["send_groups"]
                        if p["form"] == SPLIT:
                            assert sync and p["senders"] == p["send_groups"] and p["grid"] > n, what
                        else:
                            assert p["grid"] == n and p["senders"] in (p["send_groups"], p["grid"]), what
                        forms.add(p["form"])
    assert forms == ({FEW, GENERAL, WIDE} if sync == 0 else {FEW, GENERAL, SPLIT})


@pytest.mark.parametrize("sync,R,k,Tr,H,form", [
    (0, 64, 8, 128, 7168, WIDE), (0, 32, 8, 63, 7168, GENERAL), (0, 16, 8, 128, 2048, GENERAL), (0, 32, 2, 128, 7168, FEW),
    (1, 16, 8, 128, 2048, GENERAL), (1, 64, 8, 128, 7168, GENERAL),
    (1, 32, 1, 1024, 256, SPLIT), (1, 64, 8, 128, 256, SPLIT), (1, 64, 9, 128, 256, GENERAL), (1, 32, 1, 1024, 1024, FEW),
    (3, 16, 3, 700, 512, SPLIT), (3, 16, 4, 700, 512, GENERAL), (2, 16, 1, 256, 512, FEW), (2, 16, 1, 257, 512, SPLIT),
    (1, 4, 2, 128, 256, SPLIT), (1, 4, 2, 129, 256, FEW), (2, 16, 4, 2, 4992, SPLIT), (2, 8, 8, 16, 2048, GENERAL),
    (3, 64, 8, 4, 7168, SPLIT), (3, 64, 8, 8, 7168, GENERAL)])
def test_forms_of_the_one_launch_layers(geo, sync, R, k, Tr, H, form):
    """Both sides of each bound of the rule."""
    assert geo.decomposed_form(R, R * (256 // R), k, Tr, H, sync) == form


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


def chunks(geo, R, E, k, Tr):
    out = (ctypes.c_int * 8)()
    geo.layout_chunks(R, E, k, Tr, out)
    return dict(zip(("CT", "NC", "nblk", "pCT", "pNC", "pnblk", "sum", "place"), out))


def place_shapes():
    """Ranks of up to 256 x choices x tokens per rank around every place where the chunks change: one
    chunk and the longest chunks per rank, 256 and 512 chunks, powers of two and their neighbours."""
    for R in sorted({1, 2, 3, 5, 7, 8, 16, 24, 31, 32, 43, 64, 85, 86, 100, 127, 128, 129, 130, 170, 171, 172, 200, 240,
                     241, 250, 255, 256}):
        for k in (1, 2, 3, 5, 7, 8, 9, 13, 16, 22, 23, 31, 32):
            cap = 1024 // k
            around = [cap, 2 * cap, 3 * cap, 256 * cap // R, 512 * cap // R, 256 // R + 1, 61440 // R, 16384 // R]
            around += [1 << i for i in range(17)]
            for Tr in sorted({t + d for t in around for d in (-1, 0, 1)}):
                if 0 <= Tr * R * k < 1 << 31:
                    yield R, R * (256 // R), k, Tr


def test_place_kernel_chunks(geo):
    """route_place over all shapes: the chunks that are launched cover every rank's tokens, are no more than
    the workspace is sized for and fit the kernel's steps; the bound on its 16-bit sums holds for the sums
    counted chunk by chunk, and no layout is taken whose sums can reach 2^16. The bf16 layouts of at most 256
    pairs per chunk, whose row kernel writes recv_src and recv_j, are all taken."""
    taken = 0
    for R, E, k, Tr in place_shapes():
        g = chunks(geo, R, E, k, Tr)
        what = (R, E, k, Tr, g)
        assert g["pnblk"] <= g["nblk"] and g["pnblk"] == R * g["pNC"], what
        assert g["pCT"] * g["pNC"] >= Tr and g["pCT"] * k <= 1024, what
        counted = geo.place_sum_counted(R, E, k, Tr)
        assert counted <= g["sum"], what
        if g["place"]:
            taken += 1
            assert counted < 65536 and g["nblk"] <= 512, what
            share, tpw = -(-min(g["pCT"], max(Tr, 1)) // 4), 64 // k  # tokens per wave, and per step
            assert -(-share // tpw) <= (2 if g["pCT"] * k <= 256 else 6), what
        if g["CT"] * k <= 256:
            assert g["place"], what
    assert taken > 1000
    assert not chunks(geo, 257, 257, 8, 100)["place"]   # more than 256 experts
    assert chunks(geo, 1, 256, 8, 61440) == dict(CT=128, NC=480, nblk=480, pCT=128, pNC=480, pnblk=480, sum=61440, place=1)
    assert not chunks(geo, 1, 256, 8, 61441)["place"]   # 481 chunks: sums of up to 65536
    assert chunks(geo, 241, 241, 8, 130)["place"]       # longer chunks than the layout's own


@pytest.mark.parametrize("R,E,k,Tr,H,fp8,one", [
    (16, 128, 8, 128, 2048, 0, 1), (32, 160, 8, 37, 5120, 0, 1), (4, 16, 2, 128, 256, 0, 1),  # decode shapes
    (16, 128, 8, 128, 2048, 1, 0), (16, 128, 8, 64, 7168, 1, 1), (8, 64, 4, 192, 2048, 1, 1), (8, 64, 4, 256, 4096, 1, 0),
    (4, 64, 2, 704, 128, 0, 1), (4, 64, 2, 705, 128, 0, 0),    # 2816 and 2820 tokens
    (4, 64, 1, 1024, 128, 0, 1), (16, 64, 1, 257, 128, 0, 0), (2, 64, 1, 1409, 128, 0, 0),  # top-1: 4096 from four ranks on
    (4, 64, 1, 4096, 128, 0, 0), (64, 64, 2, 128, 128, 0, 0),  # where one launch took up to 1.47 times as long
    (1024, 1024, 1, 16, 512, 0, 1), (1024, 1024, 1, 16, 512, 1, 1), (512, 512, 1, 32, 128, 0, 0),  # short ranks
    (16, 64, 1, 128, 2048, 1, 1), (16, 64, 1, 129, 2048, 1, 0), (1, 8, 1, 4096, 2048, 1, 0), (8, 64, 5, 352, 128, 0, 0)])
def test_small_layers_whose_rows_go_with_the_layout(geo, R, E, k, Tr, H, fp8, one):
    """The layers that take one launch, on both sides of each bound of the rule."""
    assert geo.small_dispatch(R, E, k, Tr, H, fp8) == one


@pytest.mark.parametrize("R,k,Tr,H,workers,long", [
    (128, 8, 64, 7168, 64, 1), (64, 8, 128, 7168, 32, 1), (16, 8, 128, 2048, 32, 1),
    (128, 8, 64, 7168, 96, 0), (16, 8, 128, 2048, 48, 0), (64, 8, 64, 4096, 48, 0),  # fewer than 32 units a slice
    (256, 8, 32, 512, 8, 0), (32, 8, 64, 5120, 48, 0),  # more slices than run at once, rows in the cache
    (256, 8, 16, 1024, 64, 0), (64, 2, 64, 512, 64, 0)])
def test_scheduled_slices_form(geo, R, k, Tr, H, workers, long):
    """Both sides of each bound; the last two lost 1.3 and 1.5 times in the long form."""
    geo.long_slices.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int64]
    assert geo.long_slices(R * Tr * k, H, R * workers) == long

"""The launch planner on the CPU: plan_check.cpp compiles csrc/qlin.cpp for the
host, without kernels, and plans groups of layers of any size on a device of
256 compute units.
"""

import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2607_04244_amd import qlin

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
AUTO, GEMV, SKINNY, TILED, REGS = qlin.PATH_AUTO, qlin.PATH_GEMV, qlin.PATH_SKINNY, qlin.PATH_TILED, qlin.PATH_REGS


class Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int64) for n in ("kern", "S", "Gn", "TnMax", "rows", "ws_bytes")]


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP headers")
    so = str(tmp_path_factory.mktemp("plan") / "plan_check.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I",
                    os.path.join(ROCM, "include"), "-o", so, os.path.join(HERE, "plan_check.cpp"),
                    "-L", os.path.join(ROCM, "lib"), "-lamdhip64", "-Wl,-rpath," + os.path.join(ROCM, "lib")],
                   check=True)
    lib = ctypes.CDLL(so)
    i64 = ctypes.c_int64
    members = [ctypes.c_int, ctypes.POINTER(ctypes.c_int), ctypes.c_int]
    lib.pc_plan.argtypes = members + [ctypes.c_int, ctypes.c_int, i64, i64, i64, ctypes.POINTER(Plan)]
    lib.pc_wrong_work.argtypes = members + [ctypes.c_int, i64, i64, i64]
    lib.pc_wrong_work.restype = i64
    lib.pc_wrong_chunks.argtypes = [ctypes.c_int, i64]
    lib.pc_wrong_chunks.restype = i64
    return lib


def _members(Ns, K):
    return len(Ns), (ctypes.c_int * len(Ns))(*Ns), K


def plan(lib, Ns, K, M, path=AUTO, split=0, ws=-1, symmetric=False):
    """(status, Plan) of one launch over linears of K x N for each N."""
    p = Plan()
    rc = lib.pc_plan(*_members(Ns, K), symmetric, path, split, M, ws, ctypes.byref(p))
    return rc, p


@pytest.mark.parametrize("Ns,K,M,path,split", [
    ([1 << 20] * 8, 128, 64, SKINNY, 0),       # over 100000 ranges, no K split
    ([1048512] * 8, 128, 48, SKINNY, 0),
    ([1 << 20], 128, 64, SKINNY, 0),
    ([1 << 20] * 8, 256, 16, AUTO, 0),
    ([1 << 20] * 8, 128, 16, REGS, 0),
    ([1 << 20] * 8, 128, 4, GEMV, 0),
    ([8 * 16 * 4095], 65536, 4, REGS, 512),    # the most chunks over the most ranges
    ([256], 65536, 16, REGS, 64),
    ([16], 1024, 3, GEMV, 8),                  # one range
])
def test_every_workgroup_finds_its_chunk(planner, Ns, K, M, path, split):
    """A workgroup's chunk and range are bid / Gn and bid % Gn for every launch
    the planner accepts; a quotient one too large makes it read and write
    outside its member."""
    assert planner.pc_wrong_work(*_members(Ns, K), path, split, M, -1) == 0


def test_chunk_of_any_range_count(planner):
    for Gn in list(range(1, 300)) + [2 ** i + d for i in range(9, 22) for d in (-1, 0, 1)] + [4093, 87376, 104864, 524287]:
        assert planner.pc_wrong_chunks(Gn, min(512, (2 ** 31 - 1) // Gn)) == 0, Gn


@pytest.mark.parametrize("Ns,K,M,split", [([32768], 512, 64, 0), ([24576], 512, 50, 0), ([32768], 384, 64, 0),
                                          ([19456], 2560, 64, 0), ([26464, 400], 512, 62, 0), ([151936], 2560, 64, 0),
                                          ([20480], 896, 49, 1)])
def test_wide_layers_at_49_to_64_rows_need_no_scratch(planner, Ns, K, M, split):
    """One launch without a K split, whatever workspace there is: the launch
    without an allocation, whose scratch is 16 MiB, takes them all."""
    for ws in (-1, 0, 16 << 20):
        rc, p = plan(planner, Ns, K, M, split=split, ws=ws)
        assert rc == qlin.QLIN_OK and (p.S, p.ws_bytes, p.rows) == (1, 0, M), (ws, rc, p.S, p.ws_bytes, p.rows)


@pytest.mark.parametrize("Ns,K,M,path,split,rc,chunks,rows", [
    ([1264, 208, 292320], 6144, 27, SKINNY, 4, qlin.QLIN_ERR_UNSUPPORTED, 0, 0),   # its x and sums exceed LDS
    ([431280], 16128, 30, SKINNY, 8, qlin.QLIN_ERR_UNSUPPORTED, 0, 0),
    ([2560], 9728, 64, SKINNY, 10, qlin.QLIN_ERR_UNSUPPORTED, 0, 0),
    ([2560], 9728, 64, SKINNY, 11, qlin.QLIN_OK, 11, 64),
    ([3328, 257568, 96528, 80, 240, 96, 288, 144], 896, 35, AUTO, 4, qlin.QLIN_OK, 1, 35),   # dropped
    ([580000], 256, 20, SKINNY, 2, qlin.QLIN_OK, 2, 16),       # more ranges than counters at 8 tiles each
    ([580000], 256, 20, AUTO, 2, qlin.QLIN_OK, 2, 16),
])
def test_forced_splits_at_17_to_64_rows(planner, Ns, K, M, path, split, rc, chunks, rows):
    """What a forced split accepts is bounded by LDS for its chunk of x and its
    sums; the automatic path runs without the split instead."""
    got, p = plan(planner, Ns, K, M, path=path, split=split)
    assert got == rc, got
    if rc == qlin.QLIN_OK:
        assert (p.S, p.rows) == (chunks, rows)
        assert planner.pc_wrong_work(*_members(Ns, K), path, split, M, -1) == 0


def test_partial_sums_in_lds_spread_over_the_banks(planner):
    """The 16-byte writes and reads of the partial sums by 16 neighbouring lanes
    touch every bank once (in row order the writes would meet four to a bank)."""
    assert planner.pc_sums_conflicts(144) == 1


def test_members_of_one_route_take_its_kernel(planner):
    """Only a group of both routes (2) runs the kernels that hold both."""
    for n in (1, 2, 8):
        every = (1 << n) - 1
        assert [planner.pc_route(n, m) for m in (0, every)] == [0, 1]
        for mixed in {1, every >> 1, every & ~1} - {0, every}:
            assert planner.pc_route(n, mixed) == 2


@pytest.mark.parametrize("M,K,N,chunks", [
    (17, 2048, 256, (1,)), (32, 2048, 1024, (1,)), (48, 1152, 256, (1,)), (64, 1408, 512, (1,)), (17, 3072, 2048, (1,)),
    (17, 4352, 2560, (1,)), (64, 3072, 2048, (1,)), (64, 9728, 256, (6, 7, 8)), (48, 9728, 4096, (2, 3)),
    (64, 9728, 2560, (2, 3, 4)), (64, 2560, 19456, (1,)), (41, 2560, 12288, (1,)),
])
def test_splits_at_17_to_64_rows(planner, M, K, N, chunks):
    """Chunks of K within 5% of the fastest of 1 to 16 timed: layers of few
    groups or wide ones are not cut (2048 x 256 at 17 rows in 4 chunks took 5.8
    us, whole 4.2), deep narrow ones are."""
    rc, p = plan(planner, [N], K, M)
    assert rc == qlin.QLIN_OK and p.S in chunks, p.S


TILED_KERNEL, MID_KERNEL = 3, 4


@pytest.mark.parametrize("M,K,Ns,kern", [
    (64, 2560, [20480], MID_KERNEL), (64, 2560, [20496], TILED_KERNEL), (64, 2560, [24576], TILED_KERNEL),
    (49, 640, [22000], TILED_KERNEL), (48, 2560, [24576], MID_KERNEL), (48, 2560, [24592], TILED_KERNEL),
    (17, 2560, [32768], MID_KERNEL), (17, 512, [65552], TILED_KERNEL), (32, 1024, [40960, 8192], TILED_KERNEL),
    (64, 4096, [41200], TILED_KERNEL), (64, 2560, [151936], TILED_KERNEL), (17, 4096, [49152], MID_KERNEL),
    (33, 9728, [32784], MID_KERNEL), (64, 128, [24576], TILED_KERNEL),
])
def test_kernel_of_very_wide_layers_at_17_to_64_rows(planner, M, K, Ns, kern):
    """The faster kernel where both were timed and a workgroup each does not hold
    all columns (2560 x 20496 at 64 rows: 26.8 us in two rounds of k_mid, 17.9 as
    161 tiled blocks), without scratch and for any of it."""
    for ws in (-1, 0, 16 << 20):
        rc, p = plan(planner, Ns, K, M, ws=ws)
        assert rc == qlin.QLIN_OK and (p.kern, p.S, p.ws_bytes, p.rows) == (kern, 1, 0, M), (ws, p.kern, p.S)
    rc, p = plan(planner, Ns, K, M, path=SKINNY)      # forced, the path's own kernel
    assert rc == qlin.QLIN_OK and p.kern == MID_KERNEL


@pytest.mark.parametrize("M,K,N,ws,kern", [
    (144, 9728, 3872, -1, TILED_KERNEL), (144, 2944, 2560, -1, TILED_KERNEL), (128, 2944, 3872, -1, TILED_KERNEL),
    (97, 4096, 3872, -1, TILED_KERNEL), (96, 9728, 8192, -1, TILED_KERNEL), (128, 4096, 2560, -1, TILED_KERNEL),
    (145, 512, 2048, -1, TILED_KERNEL), (65, 2560, 6144, -1, MID_KERNEL), (129, 2560, 6144, -1, MID_KERNEL),
    (65, 1792, 256, -1, MID_KERNEL), (96, 2560, 12288, 0, MID_KERNEL), (144, 9728, 2560, 0, MID_KERNEL),
])
def test_kernel_at_65_to_144_rows(planner, M, K, N, ws, kern):
    """The faster kernel where both were timed and differ by 8% and more (9728 x
    3872 at 144 rows: 38.6 us in k_mid, 30.7 as eight K chunks of the tiled one)."""
    rc, p = plan(planner, [N], K, M, ws=ws)
    assert rc == qlin.QLIN_OK and p.kern == kern, p.kern

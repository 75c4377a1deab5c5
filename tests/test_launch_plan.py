"""Launches stay within HIP's limit of 2^32 - 1 threads on every grid whose states fit the
memory (288 GB), CPU only: the host arithmetic of csrc/fv_launch_plan.h."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2402_05193_amd", "csrc")
LIMIT = 2 ** 32


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("plan") / "plan.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    os.path.join(HERE, "launch_plan_driver.cpp"), "-o", so], check=True)
    L = ctypes.CDLL(so)
    L.plan_shortest_zchunk.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    L.plan_adjoint.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.POINTER(ctypes.c_int)]
    L.plan_adjoint.restype = ctypes.c_longlong
    return L


@pytest.mark.parametrize("shape", [(200, 1, 1), (256, 256, 256), (1, 1, 134217720), (1, 1, 134217721),
                                   (1, 1, 2 ** 31 - 1), (16, 1, 1 << 27), (40000, 40000, 1), (3000, 3000, 1000),
                                   (1, 30000, 200000), (20000, 20000, 20)])
@pytest.mark.parametrize("threads", [256, 320])
def test_stage_launch_within_limit(plan, shape, threads):
    nx, ny, nz = shape
    tiles = -(-nx // 16) * -(-ny // 16)
    z = plan.plan_shortest_zchunk(tiles, nz, threads)
    assert 1 <= z <= nz
    assert tiles * -(-nz // z) * threads < LIMIT
    assert z == 1 or tiles * -(-nz // (z - 1)) * threads >= LIMIT   # and no chunk longer than it has to be


def test_stage_launch_beyond_limit(plan):
    assert plan.plan_shortest_zchunk(1 << 25, 7, 256) == 7


@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 71, 72, 128, 129, 1000, 1024, 20500])
@pytest.mark.parametrize("periodic", [0, 1])
def test_adjoint_split(plan, n, periodic):
    """Every cell of every line in one piece of at most 64 cells (71 when the line closes on
    itself), with seven more positions in a piece, and no more positions than threads."""
    s = (ctypes.c_int * 4)()
    lines = 12345
    blocks = plan.plan_adjoint(n, periodic, lines, s)
    pieces, slots, per_group, closed = s
    assert closed == (n == 1 or (periodic and n <= 71))
    assert (pieces, slots) == (1, n) if closed else slots - 7 == -(-n // pieces) <= 64
    assert pieces == 1 or n // pieces >= 32
    assert 1 <= per_group and per_group * slots <= 256
    assert blocks == -(-lines // per_group) * pieces


@pytest.mark.parametrize("shape,periodic,launches", [((1024, 1024, 1024), 1, 2), ((20500, 20500, 1), 0, 1),
                                                     ((1290, 1290, 1290), 0, 3), ((40000, 40000, 1), 0, 2),
                                                     ((512, 512, 512), 1, 1), ((1 << 30, 1, 1), 1, 2)])
def test_adjoint_launches(plan, shape, periodic, launches):
    """Grids of up to 2.4e9 cells (three states of 40 bytes a cell in 288 GB): the block count
    in 64 bits fits the kernel's 32, in as many launches as the limit asks for."""
    s = (ctypes.c_int * 4)()
    cells = shape[0] * shape[1] * shape[2]
    total = sum(plan.plan_adjoint(n, periodic, cells // n, s) for n in shape)
    most = plan.plan_max_adjoint_blocks()
    assert most * 256 < LIMIT <= (most + 1) * 256
    assert total < LIMIT and -(-total // most) == launches
    assert cells // min(shape) < LIMIT

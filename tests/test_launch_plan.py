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

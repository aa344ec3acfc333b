"""What a launch passes in registers is what was planned (csrc/rsr_plan.h, compiled as it stands), at the ends of every range."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("start") / "start_shim.so")
    subprocess.run(["g++", "-O2", "-std=c++20", "-Wall", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2411_06360_amd", "csrc"),
                    os.path.join(ROOT, "tests", "start_shim.cpp"), "-o", so], check=True)
    f = ctypes.CDLL(so).shim_start
    f.argtypes = [ctypes.c_int64] * 4 + [ctypes.c_int] * 5 + [ctypes.POINTER(ctypes.c_int64)] * 2
    return f


@pytest.mark.parametrize("rows,all_rows,row0", [(1, 1, 0), (5003, 5003, 0), (32768, 32768, 0), (32768, 65534, 0), (32766, 65534, 32768)])
@pytest.mark.parametrize("batch", [1, 2, 65535])
@pytest.mark.parametrize("blocks", [1, 7, 1025, 3000000])
def test_words_of_a_launch(shim, rows, all_rows, row0, batch, blocks):
    launched = 0
    for vectors in (1, 2, 4):
        for cus in (8, 256, 304):
            for threads in (0, 1024):
                planned, unpacked = (ctypes.c_int64 * 9)(), (ctypes.c_int64 * 9)()
                rc = shim(rows, all_rows, row0, blocks, 8, batch, vectors, cus, threads, planned, unpacked)
                if rc < 0:
                    continue
                launched += 1
                assert rc == 0 and list(planned) == list(unpacked), (vectors, cus, threads)
    assert launched


def test_more_than_the_words_hold_is_refused(shim):
    """Vectors and workgroups have 16 bits each."""
    planned, unpacked = (ctypes.c_int64 * 9)(), (ctypes.c_int64 * 9)()
    assert shim(1024, 1024, 0, 40, 8, 65535, 1, 256, 0, planned, unpacked) == 0
    for vectors in (1, 2, 4):
        assert shim(1024, 1024, 0, 40, 8, 65536, vectors, 256, 0, planned, unpacked) < 0
    assert shim(1024, 1024, 0, 3000000, 8, 1, 1, 100000, 0, planned, unpacked) < 0

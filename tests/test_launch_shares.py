"""The workgroups of a launch (csrc/rsr_plan.h, share_of) take every column block once for every set of vectors, in equal shares."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROOM = 1 << 20


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("share") / "share_shim.so")
    subprocess.run(["g++", "-O2", "-std=c++20", "-Wall", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2411_06360_amd", "csrc"),
                    os.path.join(ROOT, "tests", "share_shim.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.shim_shares.restype = ctypes.c_int64
    lib.shim_shares.argtypes = [ctypes.c_int64] * 2 + [ctypes.c_int] * 4 + [ctypes.c_int64, ctypes.c_void_p, ctypes.c_int64]
    return lib


@pytest.mark.parametrize("vectors", [1, 2, 4])
@pytest.mark.parametrize("batch", [1, 2, 3, 5, 8, 16, 61, 255, 1023, 1025, 8191, 65535])
def test_every_block_of_every_set_once(shim, vectors, batch):
    sets = -(-batch // vectors)
    out = np.zeros((ROOM, 3), np.uint32)
    for blocks in (1, 7, 8, 9, 63, 64, 229, 256, 257, 1366, 40001):
        for cus, most, units in ((256, 4, 1), (256, 1, 9), (24, 1, 3)):
            n = shim.shim_shares(1024, blocks, batch, vectors, cus, most, units, out.ctypes.data, ROOM)
            assert n > 0, (blocks, cus)
            s = out[:n].astype(np.int64)
            assert s[:, 0].min() >= 0 and s[:, 0].max() == sets - 1
            s = s[s[:, 1] < s[:, 2]]
            sizes = s[:, 2] - s[:, 1]
            assert sizes.max() - sizes.min() <= 1
            order = np.lexsort((s[:, 1], s[:, 0]))
            s = s[order].reshape(sets, -1, 3)  # the same number of workgroups for every set
            assert (s[:, :, 0] == np.arange(sets)[:, None]).all()
            assert (s[:, 0, 1] == 0).all() and (s[:, -1, 2] == blocks).all() and (s[:, 1:, 1] == s[:, :-1, 2]).all()

"""The launch planner (csrc/rsr_plan.h), compiled as it stands behind plain C functions (tests/plan_shim.cpp)."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS, LDS = 256, 160 * 1024  # of an MI355X


class Request(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int64) for n in ("rows", "cols", "units")] + [(n, ctypes.c_int32) for n in ("k", "parts", "planes", "max_extras", "batch", "i8")] + [
        ("stream", ctypes.c_int64)]


class Answer(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int64) for n in ("grid", "lds", "vectors", "waves", "buffers", "workgroups", "end_of_lds")]


def build(folder):
    so = os.path.join(folder, "plan_shim.so")
    subprocess.run(["g++", "-O2", "-std=c++20", "-Wall", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2411_06360_amd", "csrc"),
                    os.path.join(ROOT, "tests", "plan_shim.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.shim_panels.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 3
    lib.shim_planes_per_handle.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 2
    lib.shim_product.argtypes = [ctypes.POINTER(Request), ctypes.c_int, ctypes.c_int64, ctypes.POINTER(Answer)]
    lib.shim_shared.argtypes = [ctypes.POINTER(Request), ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.POINTER(Answer)]
    return lib


def vectors_per_pass(lib, info, batch, i8, max_extras=0, shared=False):
    """How many vectors share a pass in a product of a built index (rsr_info); shared: from rsr_matvec_multi with this product alone."""
    r = Request(info.rows, info.cols, info.work_units, info.k, info.parts, 0, max_extras, batch, int(i8), info.index_bytes + info.segment_bytes)
    a = Answer()
    if shared:
        assert lib.shim_shared(ctypes.byref(r), 1, info.compute_units, LDS, ctypes.byref(a)) == 0
    else:
        assert lib.shim_product(ctypes.byref(r), info.compute_units, LDS, ctypes.byref(a)) == 0
    return a.vectors

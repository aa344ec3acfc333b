"""Helpers for the GPU parity tests: run the HIP library through its C ABI on torch device buffers."""
from __future__ import annotations

import numpy as np

import paper_2411_06360_amd as R
from tests.launch_plan import vectors_per_pass


class DeviceIndex:
    """Context manager around rsr_preprocess / rsr_destroy."""

    def __init__(self, A: np.ndarray, k: int):
        self.handle = R.rsr_preprocess(A, k)
        self.info = R.rsr_info(self.handle)

    def __enter__(self):
        return self

    def __exit__(self, *a):
        import torch

        torch.cuda.synchronize()
        R.rsr_destroy(self.handle)
        self.handle = None

    def matvec(self, v: np.ndarray) -> np.ndarray:
        """v: [batch][rows] (or [rows]) float32 or int8 host array -> host result (float32 / int32)."""
        import torch

        squeeze = v.ndim == 1
        v2 = np.ascontiguousarray(v[None, :] if squeeze else v)
        batch = v2.shape[0]
        dv = torch.from_numpy(v2).cuda()
        stream = torch.cuda.current_stream().cuda_stream
        if v2.dtype == np.float32:
            out = torch.full((batch, self.info.cols), float("nan"), dtype=torch.float32, device="cuda")
            R.rsr_matvec(self.handle, dv, out, batch, stream)
        elif v2.dtype == np.int8:
            out = torch.full((batch, self.info.cols), -(2**31), dtype=torch.int32, device="cuda")
            R.rsr_matvec_i8(self.handle, dv, out, batch, stream)
        else:
            raise TypeError(v2.dtype)
        torch.cuda.synchronize()
        res = out.cpu().numpy()
        return res[0] if squeeze else res


def assert_f32_close(got: np.ndarray, exact64: np.ndarray, v: np.ndarray, rel: float = 1e-5) -> float:
    """The stated bound: |gpu - oracle| <= rel * sum_i |v_i| for every output of every batch lane."""
    v2 = v[None, :] if v.ndim == 1 else v
    g2 = got[None, :] if got.ndim == 1 else got
    e2 = exact64[None, :] if exact64.ndim == 1 else exact64
    assert g2.shape == e2.shape
    assert np.isfinite(g2).all(), "non-finite output (an output was not written?)"
    bound = rel * np.abs(v2.astype(np.float64)).sum(axis=1, keepdims=True)
    err = np.abs(g2.astype(np.float64) - e2)
    worst = float((err / bound).max())
    assert worst <= 1.0, f"max error is {worst:.3g} x the allowed 1e-5*sum|v|"
    return worst


def batch_per_pass(planner, info, i8: bool, max_extras: int = 0) -> dict:
    """{1: .., 2: .., 4: ..}: the smallest of some batches (most of them leave a last set with fewer vectors) whose product takes a pass
    over so many vectors.  All three have to be reached."""
    found = {}
    for batch in (1, 2, 3, 5, 7, 9, 11, 13, 17, 23, 33, 49, 65, 97, 131, 195, 263, 390, 521, 1043):
        found.setdefault(vectors_per_pass(planner, info, batch, i8, max_extras), batch)
    assert set(found) == {1, 2, 4}, (found, info.rows, info.cols, info.k, info.work_units)
    return found


def batches_per_pass(planner, info, i8: bool, passes, max_extras: int = 0, shared: bool = False) -> dict:
    """{(vectors per pass, vectors of the last set if it is not full, otherwise 0): the smallest such batch}, all of them for every one of `passes`."""
    want = {(v, left) for v in passes for left in range(v)}
    found = {}
    for batch in range(1, 1200):
        v = vectors_per_pass(planner, info, batch, i8, max_extras, shared)
        found.setdefault((v, batch % v), batch)
        if want <= set(found):
            break
    assert want <= set(found), (found, info.rows, info.cols, info.k, info.work_units)
    return {key: found[key] for key in sorted(want)}


def extra_slots(planner, A: np.ndarray, k: int) -> int:
    """Further pieces (of 256 rows) of the segments of a panel, at most."""
    parts = [A == 1] + ([A == -1] if (A < 0).any() else [])
    panels = planner.shim_panels(A.shape[0], k, len(parts), 0)  # of a block: all values of both parts, or windows of one part's values
    together, windows = (len(parts), 1) if panels == 1 else (1, panels // len(parts))
    most = 0
    for c in range(0, A.shape[1], k):
        values = [P[:, c:c + k].astype(np.int64) @ (1 << np.arange(k - 1, -1, -1))[: P[:, c:c + k].shape[1]] for P in parts]
        pieces = np.array([np.maximum(0, -(-np.bincount(x, minlength=1 << k) // 256) - 1) for x in values])
        pieces[:, 0] = 0  # (value 0 is not stored)
        most = max(most, int(pieces.reshape(len(parts) // together, together, windows, -1).sum(axis=(1, 3)).max()))
    return most

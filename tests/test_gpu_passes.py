"""Passes over one, two and four vectors, from single and shared launches, where the planner's choice changes: sizes at which
a wider pass does not fit in LDS, and shared launches with units enough for the wider passes."""
import numpy as np
import pytest

import paper_2411_06360_amd as R
from oracle import dense
from tests.gpu_util import DeviceIndex

pytestmark = pytest.mark.gpu


def stream():
    import torch

    return torch.cuda.current_stream().cuda_stream


def test_int8_vectors_at_many_panels_of_a_tall_tile():
    """Ternary, k = 16, 32768 rows: 128 panels a block, whose records for two vectors do not fit in LDS beside the rows."""
    g = np.random.default_rng(401)
    A = g.integers(-1, 2, size=(32768, 1024)).astype(np.int8)
    print("tall ternary 32768x1024 k=16", flush=True)
    with DeviceIndex(A, 16) as d:
        for batch in (1, 2, 5):
            v8 = g.integers(-128, 128, size=(batch, A.shape[0]), dtype=np.int8)
            assert np.array_equal(d.matvec(v8).astype(np.int64), dense.matvec_i8(A, v8)), batch


@pytest.mark.parametrize("rows,k", [(32768, 14), (30000, 15)])
def test_int8_vectors_at_many_bit_planes_of_a_tall_tile(rows, k):
    import torch

    g = np.random.default_rng(402)
    A = g.integers(-128, 128, size=(rows, 800), dtype=np.int8)
    print(f"eight bit planes {rows}x800 k={k}", flush=True)
    h = R.rsr_qbit_preprocess(A, k, 8)
    try:
        for batch in (1, 2, 5):
            v8 = g.integers(-128, 128, size=(batch, rows), dtype=np.int8)
            out = torch.full((batch, 800), -7, dtype=torch.int32, device="cuda")
            R.rsr_qbit_matvec_i8(h, torch.from_numpy(v8).cuda(), out, batch, stream())
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().astype(np.int64), dense.matvec_i8(A, v8, qbits=8)), batch
    finally:
        torch.cuda.synchronize()
        R.rsr_qbit_destroy(h)

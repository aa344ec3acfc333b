"""Passes over one, two and four vectors, from single and shared launches, where the planner's choice changes: sizes at which
a wider pass does not fit in LDS, and shared launches with units enough for the wider passes."""
import numpy as np
import pytest

import paper_2411_06360_amd as R
from oracle import dense
from tests.gpu_util import DeviceIndex, assert_f32_close, batches_per_pass, extra_slots
from tests.launch_plan import build

pytestmark = pytest.mark.gpu


def stream():
    import torch

    return torch.cuda.current_stream().cuda_stream


def test_int8_vectors_at_many_panels_of_a_tall_tile():
    """Ternary, k = 16, 32768 rows: 128 panels a block, whose records for two vectors do not fit in LDS beside the rows; those of one
    block are kept, and a panel of the next block waits for them."""
    g = np.random.default_rng(401)
    A = g.integers(-1, 2, size=(32768, 1024)).astype(np.int8)
    print("tall ternary 32768x1024 k=16", flush=True)
    with DeviceIndex(A, 16) as d:
        for batch in (1, 2, 5):
            v8 = g.integers(-128, 128, size=(batch, A.shape[0]), dtype=np.int8)
            assert np.array_equal(d.matvec(v8).astype(np.int64), dense.matvec_i8(A, v8)), batch
        vf = g.standard_normal((3, A.shape[0])).astype(np.float32)
        got = d.matvec(vf)
        assert_f32_close(got, dense.matvec_f32(A, vf), vf)
        for _ in range(20):  # (wavefronts meet at the records in another order every time)
            assert np.array_equal(d.matvec(vf), got)


@pytest.mark.parametrize("rows,cols,k", [(32768, 300, 14), (32768, 16 * 700, 16), (28001, 911, 14), (30001, 640, 15)])
def test_records_of_one_block(rows, cols, k):
    g = np.random.default_rng(404)
    A = g.integers(-1, 2, size=(rows, cols)).astype(np.int8)
    print(f"records of one block {rows}x{cols} k={k}", flush=True)
    with DeviceIndex(A, k) as d:
        vf = g.standard_normal((2, rows)).astype(np.float32)
        assert_f32_close(d.matvec(vf), dense.matvec_f32(A, vf), vf)
        v8 = g.integers(-128, 128, size=(2, rows), dtype=np.int8)
        assert np.array_equal(d.matvec(v8).astype(np.int64), dense.matvec_i8(A, v8))


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


@pytest.mark.parametrize("shapes,batches", [
    ([(6912, 2560, 10)] * 3, (3, 4)),                     # a panel of 2048 slots: on the whole device it would be alone in LDS
    ([(4096, 2560, 11)] * 4, (4,)),
    ([(17000, 1280, 10)] * 2, (4, 9)),
    ([(1024, 3000, 8), (701, 4001, 8)], (2, 13, 62)),     # passes over two and four vectors, odd batches
    ([(1024, 3000, 8), (14336, 650, 11), (33, 500, 4)], (7, 33)),  # products that would take different passes alone
])
def test_shared_launches_with_several_vectors(shapes, batches):
    import torch

    g = np.random.default_rng(403)
    mats = [g.integers(-1, 2, size=(r, c)).astype(np.int8) for r, c, _ in shapes]
    hs = [R.rsr_preprocess(A, k) for A, (_, _, k) in zip(mats, shapes)]
    try:
        for batch in batches:
            print(f"shared launch of {shapes}, batch {batch}", flush=True)
            vf = [torch.from_numpy(g.standard_normal((batch, A.shape[0])).astype(np.float32)).cuda() for A in mats]
            v8 = [torch.from_numpy(g.integers(-128, 128, size=(batch, A.shape[0]), dtype=np.int8)).cuda() for A in mats]
            for v, dtype, one, many, exact in ((vf, torch.float32, R.rsr_matvec, R.rsr_matvec_multi, dense.matvec_f32),
                                               (v8, torch.int32, R.rsr_matvec_i8, R.rsr_matvec_multi_i8, dense.matvec_i8)):
                alone = [torch.full((batch, A.shape[1]), -7, dtype=dtype, device="cuda") for A in mats]
                both = [torch.full((batch, A.shape[1]), -9, dtype=dtype, device="cuda") for A in mats]
                for h, x, o in zip(hs, v, alone):
                    one(h, x, o, batch, stream())
                many(list(zip(hs, v, both)), batch, stream())
                torch.cuda.synchronize()
                for A, x, p, q in zip(mats, v, alone, both):
                    assert torch.equal(p, q)  # float: bit for bit
                    got, want = q.cpu().numpy(), exact(A, x.cpu().numpy())
                    if dtype is torch.int32:
                        assert np.array_equal(got.astype(np.int64), want)
                    else:
                        assert_f32_close(got, want, x.cpu().numpy())
    finally:
        torch.cuda.synchronize()
        for h in hs:
            R.rsr_destroy(h)


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("plan")))


@pytest.mark.parametrize("rows", [1, 3, 4, 5, 15, 16, 17, 1023, 4097, 5003, 9001, 16384])
def test_activations_at_any_address(planner, rows):
    """Staging in every pass: the last piece and the rows behind it, vectors that begin at every remainder of 16 bytes (an odd number of
    int8 rows, base pointers off by an element), sets of every number of vectors, from single and shared launches."""
    import torch

    g = np.random.default_rng(405)
    k, times = 6, 130
    A = g.integers(-1, 2, size=(rows, 3 * k)).astype(np.int8)
    A[0] = 1  # (at least one entry of each kind)
    A[rows - 1, ::2] = -1
    tiled = lambda x: np.tile(x, (1, times))
    h = R.rsr_preprocess(tiled(A), k)
    try:
        info, extras = R.rsr_info(h), extra_slots(planner, A, k)
        for i8, dtype, one, many, exact in ((False, torch.float32, R.rsr_matvec, R.rsr_matvec_multi, dense.matvec_f32),
                                            (True, torch.int32, R.rsr_matvec_i8, R.rsr_matvec_multi_i8, dense.matvec_i8)):
            passes = (1, 2) if not i8 and rows > 9001 else (1, 2, 4)  # (rows of four floats do not fit in LDS beyond)
            batches = set()
            for shared in (False, True):
                batches |= set(batches_per_pass(planner, info, i8, passes, extras, shared).values())
            print(f"activations at any address, {rows} rows, {'int8' if i8 else 'float'}, batches {sorted(batches)}", flush=True)
            for batch in sorted(batches):
                v = g.integers(-128, 128, size=(batch, rows), dtype=np.int8) if i8 else g.standard_normal((batch, rows)).astype(np.float32)
                want = tiled(exact(A, v))
                for off in (0, 1, 2, 3):
                    room = torch.full((off + v.size,), 77, dtype=torch.from_numpy(v).dtype, device="cuda")  # (it ends with the vectors)
                    room[off:] = torch.from_numpy(v.ravel()).cuda()
                    x = room[off:]
                    out = torch.full((2, batch, info.cols), -7, dtype=dtype, device="cuda")
                    one(h, x, out[0], batch, stream())
                    many([(h, x, out[1])], batch, stream())
                    torch.cuda.synchronize()
                    got = out.cpu().numpy()
                    assert np.array_equal(got[0], got[1]), (batch, off)
                    if i8:
                        assert np.array_equal(got[0].astype(np.int64), want), (batch, off)
                    else:
                        assert_f32_close(got[0], want, v)
    finally:
        torch.cuda.synchronize()
        R.rsr_destroy(h)

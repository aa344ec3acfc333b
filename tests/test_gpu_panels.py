"""The index in panels of ranked segments (csrc/rsr_layout.h) and the passes over one, two and four vectors, at the sizes
where they change course: panels of fewer values than a fold step reads, both parts in one panel or in several, row
counts on either side of the widths a segment may take (one lane, eight lanes, several pieces, more pieces than are fetched ahead
of the fold), odd rows and batches.  Which pass a call takes depends on how many units the launch has: the segment lengths are
repeated over so many column blocks that all three are taken, which is asserted."""
import numpy as np
import pytest

import paper_2411_06360_amd as R
from oracle import dense, steps
from tests.gpu_util import DeviceIndex, assert_f32_close, batch_per_pass, batches_per_pass, extra_slots
from tests.launch_plan import build

pytestmark = pytest.mark.gpu


def with_segments(lengths, width, seed):
    """A ternary matrix of `width` columns whose rows come in sets of equal rows of the given sizes, in random order."""
    g = np.random.default_rng(seed)
    patterns = g.integers(-1, 2, size=(len(lengths), width)).astype(np.int8)
    patterns[:, 0] = 1  # (no row is zero)
    return np.repeat(patterns, lengths, axis=0)[g.permutation(sum(lengths))]


def check_tables(d, A, k):
    for p, B in enumerate(steps.ternary_split(A) if (A < 0).any() else (A,)):
        for b, Bi in enumerate(steps.column_blocks(B, k)):
            sigma, L = R.rsr_export_block(d.handle, p, b)
            w = Bi.shape[1]
            values = Bi.astype(np.int64) @ (1 << np.arange(w)[::-1])
            assert np.array_equal(sigma, np.argsort(values, kind="stable")), (p, b)
            assert np.array_equal(L, np.concatenate([[0], np.cumsum(np.bincount(values, minlength=1 << w))])), (p, b)


def check_products(d, A, batches, seed):
    g = np.random.default_rng(seed)
    for batch in batches:
        v8 = g.integers(-128, 128, size=(batch, A.shape[0]), dtype=np.int8)
        v8[:, : A.shape[0] // 2] = -128
        v8[1:2] = -128  # (a segment of 256 such rows sums to the lowest 16-bit number)
        v8[2:3] = 127
        got = d.matvec(v8)
        assert np.array_equal(got.astype(np.int64), dense.matvec_i8(A, v8)), batch
        vf = g.standard_normal((batch, A.shape[0])).astype(np.float32)
        gf = d.matvec(vf)
        assert_f32_close(gf, dense.matvec_f32(A, vf), vf)
        for i in {0, batch // 2, batch - 1}:  # the order of additions does not depend on the vectors that share a pass
            assert np.array_equal(gf[i], d.matvec(vf[i])), (batch, i)


@pytest.mark.parametrize("k", [1, 3, 7, 8, 9, 11, 12, 13, 16])
def test_panel_shapes(k):
    g = np.random.default_rng(300 + k)
    for kind, rows, cols in (("binary", 1023, 2 * k + 1), ("ternary", 1501, 2 * k + 3), ("binary", 5, k)):
        A = (g.integers(0, 2, size=(rows, cols)) if kind == "binary" else g.integers(-1, 2, size=(rows, cols))).astype(np.int8)
        print(f"panel shapes {kind} {rows}x{cols} k={k}", flush=True)
        with DeviceIndex(A, k) as d:
            check_tables(d, A, k)
            check_products(d, A, (1, 3, 1201), 310 + k)


LENGTHS = [[1, 1, 1], [5, 6, 7, 8, 9], [47, 48, 49], [46, 46, 47, 47, 48, 95, 96], [255, 256, 257], [256] * 9, [511, 512, 513, 3],
           [3000, 1, 1, 700], [1] * 63 + [64], [1] * 65, list(range(1, 70))]


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("plan")))


@pytest.mark.parametrize("lengths", LENGTHS)
def test_segment_lengths(lengths):
    A = with_segments(lengths, 9, sum(lengths))
    print(f"segments of {lengths[:8]}.. rows: {A.shape}", flush=True)
    with DeviceIndex(A, 9) as d:
        check_tables(d, A, 9)
        check_products(d, A, (1, 2, 5), 17)
    A = np.tile(A, (1, 16))  # more blocks: more units, other passes
    with DeviceIndex(A, 9) as d:
        check_products(d, A, (301, 602), 18)


@pytest.mark.parametrize("lengths", LENGTHS)
def test_segment_lengths_in_every_pass(planner, lengths):
    A = with_segments(lengths, 9, sum(lengths))
    times = 200
    print(f"segments of {lengths[:8]}.. rows in every pass: {A.shape} x {times}", flush=True)
    g = np.random.default_rng(27)
    with DeviceIndex(np.tile(A, (1, times)), 9) as d:
        for i8 in (True, False):
            for vectors, batch in batch_per_pass(planner, d.info, i8, 2 * sum((n - 1) // 256 for n in lengths)).items():
                if i8:
                    v = g.integers(-128, 128, size=(batch, A.shape[0]), dtype=np.int8)
                    v[: batch // 2] = -128  # (a segment of 256 such rows sums to the lowest 16-bit number)
                    assert np.array_equal(d.matvec(v).astype(np.int64), np.tile(dense.matvec_i8(A, v), (1, times))), (vectors, batch)
                else:
                    v = g.standard_normal((batch, A.shape[0])).astype(np.float32)
                    got = d.matvec(v)
                    assert_f32_close(got, np.tile(dense.matvec_f32(A, v), (1, times)), v)
                    for j in (0, batch // 2, batch - 1):
                        assert np.array_equal(got[j], d.matvec(v[j])), (vectors, batch, j)


def test_more_pieces_than_are_fetched_ahead_of_the_fold():
    """32768 equal rows with entries of both signs: 128 pieces per part, in one panel."""
    A = np.tile(np.array([[1, -1, 0, 1]], np.int8), (32768, 1))
    A[5], A[77] = (0, 1, -1, 0), (-1, 0, 0, 0)
    with DeviceIndex(A, 4) as d:
        check_tables(d, A, 4)
        check_products(d, A, (1, 2, 4), 19)


@pytest.mark.parametrize("rows", [27649, 30001, 32768])
def test_tall_matrices_many_panels(rows):
    g = np.random.default_rng(rows)
    A = g.integers(-1, 2, size=(rows, 29)).astype(np.int8)
    with DeviceIndex(A, 13) as d:
        check_tables(d, A, 13)
        check_products(d, A, (1, 3), 20)


def test_infinities_and_nan_reach_only_the_columns_of_their_rows():
    g = np.random.default_rng(23)
    A = g.integers(-1, 2, size=(2000, 333)).astype(np.int8)
    v = g.standard_normal((700, 2000)).astype(np.float32)
    v[:, 3] = np.inf
    v[1::3, 11] = -np.inf
    v[::5, 1999] = np.nan
    with np.errstate(invalid="ignore"):
        want = np.zeros((700, 333))
        for r in (3, 11, 1999):  # sums of the special rows decide which outputs are not finite
            t = v[:, r].astype(np.float64)[:, None] * A[r][None, :]
            want += np.where((A[r] != 0)[None, :], np.where(np.isfinite(v[:, r])[:, None], 0.0, t), 0.0)
    with DeviceIndex(A, 10) as d:
        for batch in (1, 4, 700):
            got = d.matvec(v[:batch])
            w = want[:batch]
            assert np.array_equal(np.isnan(got), np.isnan(w))
            assert np.array_equal(got[np.isinf(w)], w[np.isinf(w)])
            assert np.isfinite(got[w == 0]).all()


@pytest.mark.parametrize("q,rows,k", [(3, 900, 12), (8, 30000, 16), (5, 2001, 13)])
def test_bit_planes_in_one_launch_or_several(q, rows, k):
    """q planes of 2^(k - 12) panels each and more: their records fit in LDS together, or the planes go out in groups."""
    import torch

    g = np.random.default_rng(q)
    A = g.integers(-(1 << (q - 1)), 1 << (q - 1), size=(rows, 21)).astype(np.int8)
    h = R.rsr_qbit_preprocess(A, k, q)
    try:
        for batch in (1, 3):
            v8 = g.integers(-128, 128, size=(batch, rows), dtype=np.int8)
            out = torch.full((batch, 21), -7, dtype=torch.int32, device="cuda")
            R.rsr_qbit_matvec_i8(h, torch.from_numpy(v8).cuda(), out, batch, torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().astype(np.int64), dense.matvec_i8(A, v8, qbits=q))
    finally:
        torch.cuda.synchronize()
        R.rsr_qbit_destroy(h)


@pytest.mark.parametrize("k", [1, 5, 6, 8, 9, 11, 12, 13])
def test_plain_step_2_over_panel_shapes(k):
    g = np.random.default_rng(500 + k)
    A = g.integers(-1, 2, size=(2 ** min(k, 12) + 37, 2 * k + 1)).astype(np.int8)
    v8 = g.integers(-128, 128, size=(3, A.shape[0]), dtype=np.int8)
    vf = g.standard_normal((3, A.shape[0])).astype(np.float32)
    print(f"plain step 2 {A.shape} k={k}", flush=True)
    with DeviceIndex(A, k) as d:
        R.rsr_set_step2(d.handle, R.RSR_STEP2_PLAIN)
        assert np.array_equal(d.matvec(v8).astype(np.int64), dense.matvec_i8(A, v8))
        assert_f32_close(d.matvec(vf), dense.matvec_f32(A, vf), vf)
        vf[1, 5] = np.inf  # reaches the columns of its row only
        got = d.matvec(vf)
        assert np.isfinite(got[[0, 2]]).all() and np.array_equal(np.isfinite(got[1]), A[5] == 0)


def test_more_panels_than_one_grid_of_the_builder_holds():
    """9000001 columns at k = 1: the index is built over ranges of column blocks (2^32 threads are a launch's limit)."""
    import torch

    g = np.random.default_rng(29)
    A = g.integers(0, 2, size=(2, 9000001)).astype(np.int8)
    print("many panels 2x9000001 k=1", flush=True)
    with DeviceIndex(A, 1) as d:
        assert d.info.segments == int((A.sum(axis=0) > 0).sum()) and d.info.stored_rows == int(A.sum())
        v8 = g.integers(-128, 128, size=(1, 2), dtype=np.int8)
        assert np.array_equal(d.matvec(v8).astype(np.int64), v8.astype(np.int64) @ A)
        vf = g.standard_normal((1, 2)).astype(np.float32)
        assert_f32_close(d.matvec(vf), vf.astype(np.float64) @ A, vf)
    torch.cuda.empty_cache()


@pytest.mark.parametrize("blocks", [63, 1024, 1025, 2049])
def test_beginnings_of_panels(blocks):
    """More panels than begin_kernel has threads, and one more or less: sizes, and the products of a matrix whose first blocks hold segments
    that are cut (extra slots) and whose others are short."""
    g = np.random.default_rng(601)
    rows, k = 300, 3
    A = g.integers(-1, 2, size=(rows, blocks * k)).astype(np.int8)
    A[:, :2 * k] = g.integers(0, 2, size=(1, 2 * k))  # segments of 300 rows
    print(f"{blocks} panels of {rows} rows, k={k}", flush=True)
    with DeviceIndex(A, k) as d:
        seen = [((A.reshape(rows, blocks, k) == part) * np.array([4, 2, 1])).sum(axis=2) for part in (1, -1)]
        assert d.info.stored_rows == sum(int((x != 0).sum()) for x in seen)
        assert d.info.segments == sum(len(np.unique((x + 8 * np.arange(blocks))[x != 0])) for x in seen)
        for batch in (1, 3):
            v8 = g.integers(-128, 128, size=(batch, rows), dtype=np.int8)
            assert np.array_equal(d.matvec(v8).astype(np.int64), dense.matvec_i8(A, v8)), batch


@pytest.mark.parametrize("kind,rows,k,steps,fill", [
    ("binary", 700, 11, 8, False), ("binary", 5000, 11, 8, True),
    ("binary", 5000, 12, 16, False), ("binary", 9000, 12, 16, True),
    ("binary", 5000, 13, 16, False), ("binary", 17000, 13, 16, True),  # panels of half a block
    ("ternary", 5000, 12, 16, False),                                  # panels of one part
])
@pytest.mark.parametrize("cut", [False, True])
def test_folds_of_two_int8_vectors(planner, kind, rows, k, steps, fill, cut):
    """Panels of one part in passes over two int8 vectors: eight and sixteen steps of a fold, slots that are cleared and absent values that are
    stored, with and without segments that are cut."""
    g = np.random.default_rng(602)
    B = (g.integers(0, 2, size=(rows, 3 * k)) if kind == "binary" else g.integers(-1, 2, size=(rows, 3 * k))).astype(np.int8)
    if cut:
        B[g.permutation(rows)[:600]] = np.tile(np.array([[1, 0, 1]], np.int8), k)
    times = 80
    tiled = lambda x: np.tile(x, (1, times))[:, :-2]  # (a narrow last block)
    extras = extra_slots(planner, B, k)
    assert (extras > 0) == cut and fill == (rows >= 2 << k)
    print(f"two int8 vectors, {kind} {rows} rows, k={k}, {extras} extra slots", flush=True)
    with DeviceIndex(tiled(B), k) as d:
        assert 1 << d.info.lo_bits == 256 * steps
        for batch in batches_per_pass(planner, d.info, True, (2,), extras).values():
            v8 = g.integers(-128, 128, size=(batch, rows), dtype=np.int8)
            v8[0], v8[-1] = -128, 127
            want = tiled(dense.matvec_i8(B, v8))
            for _ in range(2):
                assert np.array_equal(d.matvec(v8).astype(np.int64), want), batch

"""Where groups end inside a step of eight positions: segments of one length alone, of lengths that run through every
remainder of eight, of one row (a head at every other position) and of no rows (a head at every position), each with segments of eight
lanes beside them: as they come, and over so many column blocks that the planner takes the passes over one, two and four vectors of
both types, which is asserted."""
import numpy as np
import pytest

from oracle import dense
from tests.gpu_util import DeviceIndex, assert_f32_close, batch_per_pass
from tests.launch_plan import build

pytestmark = pytest.mark.gpu


def with_lengths(lengths, width, seed):
    """A binary matrix of `width` columns with one set of equal rows per entry of `lengths`, in random order."""
    g = np.random.default_rng(seed)
    values = g.permutation(np.arange(1, 1 << width))[: len(lengths)]
    rows = np.repeat(values, lengths)[g.permutation(int(sum(lengths)))]
    return ((rows[:, None] >> np.arange(width)[::-1]) & 1).astype(np.int8)


CASES = {
    "one length": lambda m: [m] * 130,
    "mixed": lambda m: [1 + (m * i) % 11 for i in range(400)],
    "wide beside": lambda m: [m] * 70 + [60 + m, 200 + m, 256, 257 + m],
    "mostly absent": lambda m: [m * 40] * 9 + [1] * 3,  # two rows per value and more: absent values are groups of no rows
}


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("plan")))


def case(kind, m):
    lengths = CASES[kind](m)
    width = 9 if len(lengths) > 300 else 8 if len(lengths) > 100 else 7
    return lengths, width, with_lengths(lengths, width, 31 * m + len(kind))


@pytest.mark.parametrize("m", range(1, 10))
@pytest.mark.parametrize("kind", sorted(CASES))
def test_group_lengths(kind, m):
    _, width, A = case(kind, m)
    A = np.concatenate([A, -A[:, ::-1]], axis=1) if m % 2 else np.tile(A, (1, 5))  # both parts, or more blocks
    print(f"patterns: {kind}, {m}: {A.shape}", flush=True)
    g = np.random.default_rng(m)
    with DeviceIndex(A, width) as d:
        for batch in (1, 2, 5, 640, 1283):
            v8 = g.integers(-128, 128, size=(batch, A.shape[0]), dtype=np.int8)
            assert np.array_equal(d.matvec(v8).astype(np.int64), dense.matvec_i8(A, v8)), batch
        vf = g.standard_normal((1283, A.shape[0])).astype(np.float32)
        whole = d.matvec(vf)
        assert_f32_close(whole, dense.matvec_f32(A, vf), vf)
        for batch in (1, 2, 5, 640):
            assert np.array_equal(d.matvec(vf[:batch]), whole[:batch]), batch


@pytest.mark.parametrize("m", range(1, 10))
@pytest.mark.parametrize("kind", sorted(CASES))
def test_group_lengths_in_every_pass(planner, kind, m):
    lengths, width, A = case(kind, m)
    if m % 2:
        A = np.concatenate([A, -A[:, ::-1]], axis=1)  # both parts
    times = 400 // A.shape[1] * 4
    print(f"patterns in every pass: {kind}, {m}: {A.shape} x {times}", flush=True)
    g = np.random.default_rng(m)
    with DeviceIndex(np.tile(A, (1, times)), width) as d:
        for i8 in (True, False):
            for vectors, batch in batch_per_pass(planner, d.info, i8, sum((n - 1) // 256 for n in lengths)).items():
                print(f"  {'int8' if i8 else 'float'}, {vectors} per pass: {batch}", flush=True)
                if i8:
                    v = g.integers(-128, 128, size=(batch, A.shape[0]), dtype=np.int8)
                    assert np.array_equal(d.matvec(v).astype(np.int64), np.tile(dense.matvec_i8(A, v), (1, times))), (vectors, batch)
                else:
                    v = g.standard_normal((batch, A.shape[0])).astype(np.float32)
                    got = d.matvec(v)
                    assert_f32_close(got, np.tile(dense.matvec_f32(A, v), (1, times)), v)
                    for j in (0, batch // 2, batch - 1):  # the sums do not depend on the pass: bit for bit
                        assert np.array_equal(got[j], d.matvec(v[j])), (vectors, batch, j)

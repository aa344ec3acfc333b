"""Where groups end inside a step of eight positions: segments of one length alone, of lengths that run through every
remainder of eight, of one row (a head at every other position) and of no rows (a head at every position), in the passes over one, two and four
vectors (small matrices, so that large batches reach the wide passes), each with segments of eight lanes beside them."""
import numpy as np
import pytest

from oracle import dense
from tests.gpu_util import DeviceIndex, assert_f32_close

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


@pytest.mark.parametrize("m", range(1, 10))
@pytest.mark.parametrize("kind", sorted(CASES))
def test_group_lengths(kind, m):
    lengths = CASES[kind](m)
    width = 9 if len(lengths) > 300 else 8 if len(lengths) > 100 else 7
    A = with_lengths(lengths, width, 31 * m + len(kind))
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

"""The launch planner (csrc/rsr_plan.h) on the host: every product that the headers admit has a launch whose LDS layout
fits, whatever the planner takes for its pass.  The planner is compiled here as it stands; the indexes are made up, with as
many units and extra slots as the builder can give them."""
import ctypes

import pytest

from tests.launch_plan import CUS, LDS, Answer, Request, build


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("plan")))


def request(shim, rows, cols, k, parts=2, planes=0, batch=1, i8=0, units_per_panel=2):
    blocks = -(-cols // k)
    units = blocks * shim.shim_panels(rows, k, parts, planes) * units_per_panel
    extras = rows * (1 if planes or parts == 1 else 2) // 256 if units_per_panel > 1 else 0
    return Request(rows, cols, units, k, parts, planes, extras, batch, i8)


def check(a, what):
    assert a.lds <= LDS and a.end_of_lds <= a.lds, what
    assert 1 <= a.waves <= 16 and a.grid >= a.workgroups >= 1 and a.buffers >= 1, what


def product(shim, *args, **kw):
    r, a = request(shim, *args, **kw), Answer()
    rc = shim.shim_product(ctypes.byref(r), CUS, LDS, ctypes.byref(a))
    assert rc == 0, (rc, args, kw)
    check(a, (args, kw))
    return a


def shared(shim, requests):
    n = len(requests)
    r, a = (Request * n)(*requests), (Answer * n)()
    what = [(x.rows, x.cols, x.k, x.parts, x.batch, x.i8) for x in requests]
    assert shim.shim_shared(r, n, CUS, LDS, a) == 0, what
    for x in a:
        check(x, what)
    assert len({x.vectors for x in a}) == 1
    return a


ROWS = (1, 17, 1024, 5003, 8191, 12288, 16384, 20000, 24577, 27648, 27649, 30000, 30642, 30643, 32767, 32768)


@pytest.mark.parametrize("k", range(1, 17))
@pytest.mark.parametrize("i8", [0, 1])
def test_every_product_has_a_launch(shim, k, i8):
    for rows in ROWS:
        for parts, planes in [(1, 0), (2, 0)] + [(0, shim.shim_planes_per_handle(rows, k, q)) for q in (2, 4, 8)]:
            for blocks in (1, 7, 300, 3000):
                for batch in (1, 2, 3, 4, 16, 1201, 65535):
                    for per_panel in (1, 4):
                        product(shim, rows, blocks * k, k, parts, planes, batch, i8, per_panel)


@pytest.mark.parametrize("rows,cols,k,parts,planes", [(30643, 1024, 16, 2, 0), (32768, 1024, 16, 2, 0), (32768, 1024, 14, 0, 8), (30000, 1024, 15, 0, 8)])
def test_two_int8_vectors_share_a_pass_only_where_their_records_fit(shim, rows, cols, k, parts, planes):
    """Records of a block's panels are as many words per vector as there are panels: with 128 panels two vectors' do not fit."""
    for batch in (2, 3, 8):
        assert product(shim, rows, cols, k, parts, planes, batch, 1).vectors == 1
    assert product(shim, 16384, 16384, 12, 1, 0, 8, 1).vectors == 2  # (and where they do, they share one)


@pytest.mark.parametrize("rows,cols,k,n,batches,i8", [
    (6912, 2560, 10, 3, (3, 4), 0), (4096, 2560, 11, 4, (4,), 0), (17000, 2560, 10, 2, (4,), 1), (14336, 2816, 11, 2, (2,), 0)])
def test_a_shared_launch_takes_passes_that_fit_on_its_share(shim, rows, cols, k, n, batches, i8):
    """On the whole device a workgroup has one block here, whose panel is alone in LDS; on a share it has several."""
    for batch in batches:
        for per_panel in (4, 6, 9, 14, 20):
            shared(shim, [request(shim, rows, cols, k, 2, 0, batch, i8, per_panel)] * n)


@pytest.mark.parametrize("i8", [0, 1])
def test_every_shared_launch_fits(shim, i8):
    kinds = [(64, 4, 1), (1024, 8, 2), (2560, 10, 2), (5003, 11, 2), (6912, 10, 2), (14336, 11, 2), (16384, 12, 1), (24577, 13, 2), (30643, 16, 2), (32768, 16, 2)]
    for a in kinds:
        for b in kinds:
            for blocks in (1, 40, 256, 1500):
                for n in (2, 3, 8):
                    for batch in (1, 2, 3, 4, 7, 16, 400):
                        for per_panel in (1, 5):
                            make = lambda x, m: request(shim, x[0], m * x[1], x[1], x[2], 0, batch, i8, per_panel)
                            shared(shim, [make(a, blocks)] + [make(b, 256)] * (n - 1))


@pytest.mark.parametrize("i8", [0, 1])
@pytest.mark.parametrize("batch", [1, 2, 3, 5, 6, 7, 9, 11, 13, 16])
def test_a_launch_is_one_round_of_workgroups(shim, batch, i8):
    """A workgroup more than the device holds at a time is a second round for all."""
    for rows, k, parts in [(1024, 8, 1), (2048, 9, 2), (2902, 9, 2), (5003, 11, 2), (8265, 9, 1), (16384, 12, 1), (32768, 13, 2)]:
        for blocks in (64, 229, 300, 747, 911, 1821, 3000):
            for per_panel in (1, 2, 3, 5):
                a = product(shim, rows, blocks * k, k, parts, 0, batch, i8, per_panel)
                per_cu = min(2 if a.waves == 5 else 16 // a.waves, LDS // a.lds, 4)  # (five wavefronts: two workgroups, measured)
                assert a.grid <= CUS * per_cu, (rows, blocks, per_panel, a.waves, a.grid)


@pytest.mark.parametrize("i8", [0, 1])
def test_small_panels_do_not_count_as_lack_of_room(shim, i8):
    """Eight panels in flight are the most there can be: with a unit per panel that is no reason to take narrow passes."""
    assert product(shim, 1472, 30464, 8, 1, 0, 11, i8, 1).vectors == 4
    assert product(shim, 1024, 9881, 9, 1, 0, 2, i8, 1).vectors == 1  # (few units: a vector per pass)


@pytest.mark.parametrize("i8", [0, 1])
def test_workgroups_share_the_lds_in_pieces_of_1280_bytes(shim, i8):
    """Three workgroups of just under a third of the LDS do not fit: those that are planned would wait for a second round."""
    for rows in range(1000, 30000, 13):
        for k, batch in ((9, 8), (11, 11), (11, 2), (12, 3)):
            a = product(shim, rows, 115 * k, k, 1, 0, batch, i8, 4)
            per_cu = min(16 // a.waves, LDS // (-(-a.lds // 1280) * 1280))
            assert a.grid <= CUS * per_cu, (rows, k, batch, a.lds, a.grid)


@pytest.mark.parametrize("rows,cols,k,parts,units,batch,i8,vectors", [
    (4868, 19245, 11, 1, 5618, 11, 0, 2),    # 41 us with one vector per pass, 27 with two
    (4608, 14028, 11, 1, 3932, 11, 0, 2),    # 31 and 21
    (4901, 21824, 11, 2, 13891, 11, 0, 2),   # 94 and 68
    (5056, 26112, 10, 2, 13878, 64, 1, 4),   # 215 with two, 154 with four
    (10402, 70, 6, 2, 120, 64, 0, 2),        # 13.6 with one, 8.7 with two
    (16867, 47, 8, 2, 100, 64, 0, 2),        # 20.0 and 10.4
    (12587, 1596, 11, 1, 881, 300, 0, 2),    # 167 and 116
    (72, 9720, 11, 1, 884, 300, 0, 2),       # 215 and 161
    (23987, 3427, 13, 1, 3634, 11, 1, 2),    # 33.0 and 23.6
    (4744, 249, 14, 1, 72, 64, 1, 2),        # 16.3 and 11.6
    (3912, 71, 16, 1, 80, 64, 1, 2),         # 16.1 and 11.3
])
def test_the_pass_that_was_measured_to_be_shortest(shim, rows, cols, k, parts, units, batch, i8, vectors):
    """Units as the builder gives them; workgroups of several rounds, of few block ranges, of panels that wait for room."""
    r, a = Request(rows, cols, units, k, parts, 0, 64, batch, i8), Answer()
    assert shim.shim_product(ctypes.byref(r), CUS, LDS, ctypes.byref(a)) == 0
    check(a, (rows, cols, k))
    assert a.vectors == vectors


@pytest.mark.parametrize("rows,cols,k,parts,units,stream,batch,vectors", [
    (9645, 9664, 10, 2, 8821, 45894400, 7, 4),    # 21.4 us with two vectors per pass, 17.7 with four
    (8754, 5219, 9, 2, 5043, 24705024, 12, 4),    # 19.0 and 16.1
    (12358, 7360, 10, 2, 9489, 43555072, 7, 4),   # 20.7 and 17.7
    (2558, 2560, 10, 2, 993, 4136448, 12, 4),     # 9.1 and 7.8
    (2559, 2560, 11, 2, 700, 3267072, 7, 2),      # 8.5 with one, 7.2 with two
    (3133, 8872, 9, 2, 3944, 18285568, 2, 2),     # 8.8 and 7.6
    (4537, 1472, 9, 1, 451, 1890048, 11, 2),      # 7.3 and 6.3
    (5374, 1624, 10, 1, 514, 2267648, 2, 1),      # 4.6 with one, 5.3 with two
])
def test_int8_rows_that_are_no_multiple_of_four(shim, rows, cols, k, parts, units, stream, batch, vectors):
    """Such rows are staged as wide as others: they do not make several vectors per pass dear."""
    r, a = Request(rows, cols, units, k, parts, 0, 64, batch, 1, stream), Answer()
    assert shim.shim_product(ctypes.byref(r), CUS, LDS, ctypes.byref(a)) == 0
    check(a, (rows, cols, k))
    assert a.vectors == vectors

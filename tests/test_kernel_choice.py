"""Which kernel or form a size takes (host code only; the functions are the library's own, not part of the C ABI).  A size on
the wrong side of one of these lines still answers rightly and only gets slower, which no parity test would notice."""
import ctypes as C

import pytest

from paper_2112_13509_amd import binding as ab
from paper_2112_13509_amd import workloads as wl


def _fn(symbol, restype, *argtypes):
    f = getattr(ab.load(), symbol)
    f.restype, f.argtypes = restype, argtypes
    return f


@pytest.mark.parametrize("S,Cn,vec,lanes", [
    (1, 128, True, 16), (65536, 128, False, 16), (1, 129, False, 64), (4096, 256, True, 64), (4097, 256, True, 16),
    (65536, 256, False, 16), (8192, 257, False, 64), (8193, 320, False, 16), (65536, 321, False, 64),
    (1, 512, True, 64), (65536, 512, True, 16), (64, 513, False, 64), (1, 1024, True, 64), (65536, 1024, True, 64)])
def test_lanes_of_a_decision_row(S, Cn, vec, lanes):
    """Sixteen lanes a row made a decision on few long rows twice as long (1024 columns: 3.8 -> 7.6 us)."""
    assert _fn("_ZN2ab12decide_lanesElib", C.c_int, C.c_int64, C.c_int, C.c_bool)(S, Cn, vec) == lanes


@pytest.mark.parametrize("hidden,S,Cn,kernel", [
    ((128, 1280), 512, 256, 1), ((128, 1280), 64, 512, 1), ((128, 2048, 256), 256, 256, 1),     # two slabs of inputs
    ((128, 1280), 512, 255, 0), ((128, 1280), 8, 256, 0),                                       # tiles that span scenarios; few tiles
    ((128, 1024), 512, 256, 1), ((128, 1024), 512, 255, 2), ((192, 1280), 512, 256, 1), ((64, 1280), 512, 256, 1), ((1088, 1280), 64, 256, 1)])
def test_kernel_of_the_first_hidden_product(hidden, S, Cn, kernel):
    """128 inputs and more than 1024 outputs had fallen to the generic tiles (128-2048-256, 256 scenarios: 136 -> 333 us a call)."""
    d = ab.desc_from_workload(wl.make_scoring("kernel-choice", 1, 4, list(hidden), 4, 4, 16e3, 64e6, 1.0, 16.0, False, "bf16", 1))
    assert _fn("_ZN2ab18scoring_big_kernelEPK13ab_model_desclii", C.c_int, C.c_void_p, C.c_int64, C.c_int32, C.c_int)(C.byref(d), S, Cn, 1) == kernel


@pytest.mark.parametrize("hidden,Cn,k,first", [
    ((512, 512), 256, 1, 6), ((1024, 1024), 256, 1, 3), ((1024, 256), 255, 1, 12), ((256, 256), 256, 1, 40), ((128, 1024), 256, 1, 10),
    ((512, 512, 512), 256, 1, 18), ((512, 512, 512), 256, 2, 18), ((1024,) * 4, 256, 2, 11), ((1024,) * 4, 255, 1, 11), ((256, 256, 256), 256, 1, 64),
    ((512, 1280), 256, 1, 13), ((1024, 512, 256), 256, 2, 36),
    # inputs that the streaming generating kernel does not take (2048-256, 12 scenarios on whole tiles: 47.7 -> 62.4 us a call)
    ((2048, 256), 256, 1, 64), ((1280, 512), 256, 1, 32), ((2048, 1024), 256, 1, 16), ((64, 256), 256, 1, 64), ((64, 1024), 256, 1, 16),
    ((1280, 512, 256), 256, 1, 32), ((2048, 1024, 1024), 256, 1, 16), ((2048, 1024, 1024), 256, 2, 16),
    # behind generic tiles (256-512-512, 18 scenarios 24.7 -> 26.4 us a call), and wide ones in front of them (512-768-192, 12 scenarios 28.4 -> 30.3)
    ((256, 512, 512), 256, 2, 32), ((256, 640, 256), 256, 2, 64), ((256, 768, 256), 256, 2, 36), ((256, 1024, 1024), 256, 2, 16), ((256, 768, 512), 256, 2, 22),
    ((1024, 1280, 256), 260, 2, 63), ((768, 2048, 512), 256, 2, 26), ((512, 768, 192), 256, 1, 22), ((512, 768, 64), 256, 1, 12), ((512, 768, 256), 256, 1, 22), ((768, 1024, 256), 256, 1, 13),
    ((1024, 1024, 192), 256, 1, 13), ((512, 512, 192), 256, 1, 18), ((768, 1024, 1024, 192), 256, 2, 13), ((1280, 1280, 1024, 192), 256, 2, 16),
    ((512, 768, 512), 256, 1, 18), ((128, 512), 255, 1, 24), ((128, 512), 260, 1, 19)])
def test_fewest_tiles_of_the_large_kernels(hidden, Cn, k, first):
    """From so many scenarios on (parts of tiles fill the chip; 1024-1024, 14 scenarios on generic tiles: 23.1 -> 32.9 us a call), and a
    workspace that holds the other kernels' partial sums below."""
    f = _fn("_ZN2ab18scoring_big_kernelEPK13ab_model_desclii", C.c_int, C.c_void_p, C.c_int64, C.c_int32, C.c_int)
    d = ab.desc_from_workload(wl.make_scoring("kernel-choice", 1, 4, list(hidden), 4, 4, 16e3, 64e6, 1.0, 16.0, False, "bf16", 1))
    assert [f(C.byref(d), S, Cn, k) > 0 for S in (first - 1, first, 300)] == [False, True, True]
    if -(-first * Cn // 256) * (hidden[k] // 256) < 64:
        sizes = [ab.ab_workspace_bytes(d, S, Cn, 0) for S in range(max(1, first - 3), first + 4)]
        assert sizes == sorted(sizes)


@pytest.mark.parametrize("hidden,S,Cn,k,parts", [
    # on 256 and on 304 CUs: 8 of an XCD's 32 or 38 work-groups hold quarters, 16 (19) halves
    ((512, 1024), 13, 256, 1, (4, 4)), ((512, 1024), 17, 256, 1, (2, 2)), ((512, 1024), 33, 256, 1, (1, 1)), ((1024, 1024, 1024), 64, 256, 2, (1, 1)),
    ((1024, 1024, 1024), 72, 256, 2, (4, 1)), ((1024, 1024, 1024), 80, 256, 1, (4, 4)), ((1024, 1024, 1024), 96, 255, 1, (2, 2)), ((1024, 1024, 1024), 300, 256, 2, (1, 1)),
    # not a streaming kernel; more than four column tiles
    ((2048, 256), 100, 256, 1, (0, 0)), ((512, 256), 4, 256, 1, (0, 0)), ((128, 1280), 512, 256, 1, (1, 1))])
def test_parts_of_the_last_round_of_tiles(hidden, S, Cn, k, parts):
    """Whole tiles leave work-groups idle there (1024 four times, 16 scenarios: 59 -> 76 us a call)."""
    f = _fn("_ZN2ab22scoring_parts_of_tilesEPK13ab_model_descliii", C.c_int, C.c_void_p, C.c_int64, C.c_int32, C.c_int, C.c_int)
    d = ab.desc_from_workload(wl.make_scoring("kernel-choice", 1, 4, list(hidden), 4, 4, 16e3, 64e6, 1.0, 16.0, False, "bf16", 1))
    assert tuple(f(C.byref(d), S, Cn, k, cus) for cus in (256, 304)) == parts


@pytest.mark.parametrize("hidden,S,Cn,groups", [
    ((256, 256), 1024, 4096, [1]), ((256, 256), 96, 128, [2]), ((256, 256), 95, 128, [0]), ((64, 64), 192, 128, [1]), ((64, 64), 191, 128, [0]),
    ((256, 128, 64), 192, 128, [1, 1]), ((256, 128, 64), 191, 128, [0, 0]), ((64, 512, 64), 48, 128, [4, 0]), ((256, 256), 4, 4096, [2]), ((256, 256), 4, 512, [0]),
    # wide last layers: groups enough for the chip
    ((64, 4096), 8, 1024, [8]), ((64, 4096), 64, 1024, [1]), ((64, 4096), 130, 1024, [8]), ((64, 4096), 520, 1024, [2]), ((64, 4096), 1024, 1024, [1]),
    ((64, 1280), 130, 1024, [5]), ((64, 768), 50, 1024, [1]), ((64, 768), 75, 1024, [3]), ((256, 1024, 1024), 64, 1024, [8, 1])])
def test_fp32_products_on_the_bf16_matrix_cores(hidden, S, Cn, groups):
    """From 192 tiles on (128-128 with 16000 rows, 124 tiles: 22.7 -> 23.5 us a call); the last layer's column tiles in one group only where
    the rows fill the chip (64-4096 with 8192 rows: 59 -> 125 us)."""
    f = _fn("_ZN2ab20scoring_split_groupsEPK13ab_model_desclii", C.c_int, C.c_void_p, C.c_int64, C.c_int32, C.c_int)
    d = {t: ab.desc_from_workload(wl.make_scoring("kernel-choice", 1, 4, list(hidden), 4, 4, 16e3, 64e6, 1.0, 16.0, False, t, 1)) for t in ("f32", "bf16")}
    assert [f(C.byref(d["f32"]), S, Cn, k) for k in range(1, len(hidden))] == groups
    assert not any(f(C.byref(d["bf16"]), S, Cn, k) for k in range(1, len(hidden)))


@pytest.mark.parametrize("dtype,L,hidden,last", [
    ("bf16", 128, (1024, 1024), 112), ("bf16", 133, (1024, 1024), 64), ("bf16", 100, (512, 512), 224), ("bf16", 128, (64, 64), 1792),
    # long rows: by units, scenarios and the kind of logarithm
    ("bf16", 1132, (64, 64), 1024), ("bf16", 1133, (64, 64), 0), ("bf16", 1136, (64, 64), 0), ("bf16", 1300, (64, 64), 0), ("bf16", 497, (64, 64), 1024),
    ("bf16", 499, (64, 64), 0), ("bf16", 601, (512, 64), 128), ("bf16", 1001, (512, 64), 0), ("bf16", 1360, (512, 64), 128), ("bf16", 1364, (1024, 64), 64),
    ("bf16", 1365, (1024, 64), 0), ("f32", 128, (256, 256), 2048), ("f32", 128, (64, 64), 8192), ("f32", 341, (64, 64), 16),
    ("f32", 300, (64, 64), 16), ("f32", 300, (512, 64), 1024)])
def test_scenario_term_in_the_first_launch(dtype, L, hidden, last):
    """Few scenarios (300 of 534 columns, 512 units in bf16, joined: 36.4 -> 40.4 us a call) and rows that are not too long for the
    tiles that there are (4096 columns, 64 units in bf16: 17.7 -> 22.1)."""
    f = _fn("_ZN2ab20term_in_first_launchEPK13ab_model_descl", C.c_bool, C.c_void_p, C.c_int64)
    d = ab.desc_from_workload(wl.make_scoring("kernel-choice", 1, L, list(hidden), 4, 4, 16e3, 64e6, 1.0, 16.0, False, dtype, 1))
    assert [f(C.byref(d), S) for S in (max(last, 1), last + 1)] == [last > 0, False]


@pytest.mark.parametrize("dtype,hidden,S,Cn,joined", [
    ("bf16", (512,), 4, 1024, [True, True]), ("bf16", (512,), 4, 1025, [False, True]), ("f32", (512,), 4, 3072, [True, True]),
    ("f32", (512,), 4, 3073, [False, True]), ("bf16", (1024, 64), 4, 4096, [False, True]), ("bf16", (1024, 64), 1, 4096, [True, True]),
    ("f32", (1024, 64), 4, 4096, [False, True]), ("f32", (1024, 64), 16, 4096, [True, True])])
def test_opening_with_a_large_candidate_table(dtype, hidden, S, Cn, joined):
    """Shared grid and a grid per scenario (which has no table).  Beside the scenario term's blocks the table's run slower (1024 x 4096 in
    bf16, one scenario: 34.7 -> 50.4 us a call)."""
    f = _fn("_ZN2ab22scoring_joined_openingEPK13ab_model_desclii", C.c_bool, C.c_void_p, C.c_int64, C.c_int32, C.c_int)
    d = ab.desc_from_workload(wl.make_scoring("kernel-choice", 1, 64, list(hidden), 4, 4, 16e3, 64e6, 1.0, 16.0, False, dtype, 1))
    assert [f(C.byref(d), S, Cn, own) for own in (0, 1)] == joined


def _update_desc(dtype, L, hidden, n=0):
    return ab.desc_from_workload(wl.make_update(N=64, batch=64, L=L, hidden=hidden, dtype=dtype, n_workers=n))


def takes_rows(d, B, first=0):
    return _fn("_ZN2ab17update_takes_rowsEPK13ab_model_descli", C.c_bool, C.c_void_p, C.c_int64, C.c_int)(C.byref(d), B, first)


def rows32(d, first=0):
    return _fn("_ZN2ab13update_rows32EPK13ab_model_desci", C.c_int, C.c_void_p, C.c_int)(C.byref(d), first)


@pytest.mark.parametrize("dtype,L,hidden,first,rows,layers", [
    # light: the row-block form at every batch
    ("bf16", 128, (512, 512, 512), 0, (1, 4096, 5000, 1 << 20), ()), ("bf16", 128, (1024, 512, 256), 0, (1, 4097), ()),
    ("bf16", 128, (512, 1024), 0, (64, 9000), ()), ("f32", 64, (256, 256), 0, (64, 9000), ()), ("f32", 128, (512, 256), 0, (64,), ()),
    # heavy: where the blocks fill the chip
    ("bf16", 128, (1024, 1024), 0, (3072, 4096, 6144, 8193), (64, 512, 3071, 4097, 6143)),
    ("bf16", 128, (1024,), 0, (3072, 65536), (1, 1024)), ("bf16", 128, (640, 640, 640), 0, (4096,), (1024, 5000)),
    ("f32", 128, (512, 512), 0, (3072, 7168, 8193), (64, 3071, 6144)), ("f32", 64, (448, 448), 0, (4096,), (2048, 4097, 8192, 65536)),
    # frozen layers shorten the stream
    ("bf16", 128, (768, 768), 1, (512, 2048), ()), ("bf16", 128, (1024,), 1, (64, 2048), ()), ("f32", 128, (384, 384), 2, (), (64, 512)),
    # output unit alone: large batches of light networks layer by layer (198-256-128-64-1 in bf16, 60000 rows: 152 -> 185 us)
    ("f32", 64, (256, 128, 64), 3, (64, 24576), (24577, 1 << 20)), ("bf16", 64, (256, 128, 64), 3, (16384,), (16385,)),
    ("f32", 64, (256, 128, 64), 2, (65536,), ()), ("bf16", 64, (256, 256), 2, (64, 65536), ()), ("f32", 64, (256,), 1, (65536,), ()),
    # beyond the row-block form's widths, weights or LDS
    ("bf16", 8, (1088, 64), 0, (), (64, 4096)), ("bf16", 30, (1024, 1024, 1024), 0, (), (64, 4096)), ("f32", 4, (1024, 512), 0, (), (64, 8193))])
def test_form_of_an_update_step(dtype, L, hidden, first, rows, layers):
    """The row-block form had taken every network that it can take, at 1.1 to 1.3 times the time of the layer-by-layer form for
    heavy ones at small batches (390-1024-1024-1 in bf16, 512 rows: 71 -> 92 us)."""
    d = _update_desc(dtype, L, hidden)
    assert [takes_rows(d, B, first) for B in rows + layers] == [True] * len(rows) + [False] * len(layers)


def gradient_plan(d, B, first=0):
    """Tile width, batch shares of the tiles and of the output unit; zeros where a step has no gradient launch of its own."""
    f = _fn("_ZN2ab20update_gradient_planEPK13ab_model_desclii", C.c_int, C.c_void_p, C.c_int64, C.c_int, C.c_int)
    return tuple(f(C.byref(d), B, first, what) for what in range(3))


@pytest.mark.parametrize("dtype,L,hidden,n,first,B,plan", [
    ("f32", 16, (64, 64), 0, 0, 1024, (0, 0, 0)), ("f32", 16, (64, 64), 0, 0, 1025, (64, 8, 8)), ("f32", 16, (64, 64), 0, 0, 4032, (64, 8, 8)),
    ("f32", 16, (64, 64), 0, 0, 4096, (64, 16, 16)), ("f32", 16, (64, 64), 0, 0, 65536, (64, 64, 64)), ("bf16", 16, (64,), 16, 0, 1 << 20, (64, 64, 64)),
    ("bf16", 128, (512, 512, 512), 0, 0, 4096, (0, 0, 0)), ("bf16", 128, (512, 512, 512), 0, 0, 4097, (128, 8, 8)), ("bf16", 128, (512, 512, 512), 0, 0, 8192, (128, 8, 8)), ("bf16", 128, (512, 512, 512), 8, 2, 65536, (128, 8, 32)),
    ("f32", 64, (256, 256), 0, 0, 65536, (64, 8, 16)),
    ("bf16", 16, (256, 256), 0, 0, 8192, (64, 8, 16)), ("bf16", 16, (256, 256), 0, 0, 16384, (64, 16, 16)), ("f32", 4, (1024, 512), 0, 0, 64, (0, 0, 0))])
def test_shares_of_the_batch_in_the_gradient_launch(dtype, L, hidden, n, first, B, plan):
    """Eight shares whatever the batch had left small networks on a few work-groups (54-64-16 in bf16, 65536 rows: 408 -> 522 us)."""
    assert gradient_plan(_update_desc(dtype, L, hidden, n), B, first) == plan


def one_step(d, B, first=0):
    return _fn("_ZN2ab15update_one_stepEPK13ab_model_descli", C.c_bool, C.c_void_p, C.c_int64, C.c_int)(C.byref(d), B, first)


@pytest.mark.parametrize("dtype,L,hidden,first,last", [
    ("bf16", 128, (256, 256), 0, 1024), ("bf16", 128, (512, 512), 1, 1536), ("bf16", 128, (512, 512), 0, 1536), ("bf16", 128, (512, 512, 512), 0, 4096),
    ("bf16", 128, (512, 512, 512), 3, 2048), ("bf16", 128, (1024, 512, 256), 0, 2048), ("f32", 16, (64, 64), 0, 1024), ("f32", 120, (256, 256), 0, 2048),
    ("f32", 128, (512, 256), 0, 1024)])
def test_gradients_and_adam_in_one_launch(dtype, L, hidden, first, last):
    """One launch for few rows (54-64-64-1 in fp32, 200 rows: 28.8 -> 23.6 us a step), two for many (126-64-64-1, 8192 rows: 47.5, in one 82.4)."""
    d = _update_desc(dtype, L, hidden)
    assert [one_step(d, B, first) for B in (1, last, last + 1, 16384)] == [True, True, False, False]


@pytest.mark.parametrize("dtype,L,hidden", [("bf16", 128, (1024, 1024)), ("f32", 128, (512, 512)), ("f32", 64, (448, 448)), ("bf16", 128, (1024,)),
                                            ("bf16", 20, (64, 64)), ("bf16", 30, (1024, 1024, 1024)), ("f32", 64, (256, 128, 64))])
def test_update_workspace_grows_with_the_batch(dtype, L, hidden):
    """A workspace made for the largest minibatch serves every smaller one, whichever form that takes."""
    d = _update_desc(dtype, L, hidden)
    sizes = [ab.ab_workspace_bytes(d, 0, 0, B) for B in (1, 64, 65, 200, 512, 1024, 2048, 3071, 3072, 4096, 4097, 6143, 6144, 8192, 8193, 16384, 65536)]
    assert sizes[0] > 0 and sizes == sorted(sizes)

"""fp32 products on the bf16 matrix cores (csrc/gemm_split.hip): row counts off the 128-row tile, column tiles of 128 and 64,
two slabs and many, generated and loaded operand, stored result and fused output unit, one work-group for all column tiles
and one for each, grids per scenario; each against the fp64 oracle.  Infinite and NaN statistics come out as the oracle has them."""
import ctypes as C

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2112_13509_amd import binding as ab
from paper_2112_13509_amd import workloads as wl
from gpu_helpers import Scorer
from helpers import oracle_model

pytestmark = pytest.mark.gpu


def groups(w, S, k):
    f = ab.load()._ZN2ab20scoring_split_groupsEPK13ab_model_desclii
    f.restype, f.argtypes = C.c_int, (C.c_void_p, C.c_int64, C.c_int32, C.c_int)
    return f(C.byref(ab.desc_from_workload(w)), S, w.C, k)


@pytest.mark.parametrize("S,L,P,Q,hidden,own_grids,want", [
    (97, 16, 16, 17, [64, 64], False, [1]),                # 26384 rows: 16 short of a tile
    (300, 5, 13, 7, [128, 192], False, [3]),               # three column tiles of 64
    (25, 40, 32, 32, [192, 128, 320], False, [1, 5]),      # stored and loaded activations, whole tiles
    (8, 128, 61, 7, [256, 1024], False, [8]),              # eight column tiles
    (49, 9, 16, 16, [256, 256, 256], True, [2, 2]),
    (1100, 8, 12, 11, [64, 256], False, [1]),              # one work-group walks both column tiles
    (5000, 3, 5, 9, [64, 128, 256, 64], True, [1, 2, 1]),  # scenarios of 45 candidates
    (6, 20, 64, 33, [1088, 512], True, [4]),
])
def test_split_products(S, L, P, Q, hidden, own_grids, want):
    w = wl.make_scoring("split-shapes", S, L, hidden, P, Q, 16 * wl.KIB, 64 * wl.MIB, 1.0, 64.0, False, "f32", 11000 + S)
    assert [groups(w, S, k) for k in range(1, len(hidden))] == want
    part = cred = None
    if own_grids:
        rng = np.random.default_rng(S)
        part = (w.part[None] * np.exp2(rng.uniform(-1, 1, (S, 1)))).astype(np.float32)
        cred = (w.cred[None] * rng.uniform(1, 1.25, (S, 1))).astype(np.float32)
    scores, idx, best = Scorer(w).run(part=part, cred=cred)
    ref = orc.score(oracle_model(w), w.dyn, w.scal, w.part if part is None else part, w.cred if cred is None else cred)
    # fp32 sums of up to a thousand terms: 2 to 5e-7; without one of the three smallest partial products at least 2e-6
    # (one of them is about 2^-17 of a term, the sums of their random signs likewise of the result)
    assert np.linalg.norm(scores - ref) <= 1e-6 * np.linalg.norm(ref)
    assert np.array_equal(idx, np.argmax(scores, axis=1)) and np.array_equal(best, scores[np.arange(S), idx])


@pytest.mark.parametrize("hidden", [[128, 128], [128, 128, 256], [64, 64]])
def test_infinite_and_nan_statistics(hidden):
    """All weights positive: an infinite statistic makes every score of its scenario +inf, which parts of an infinity alone
    would turn into NaN; rows of other scenarios in the same tile keep their precision."""
    S, L, P, Q = 300, 8, 13, 7
    w = wl.make_scoring("split-inf", S, L, hidden, P, Q, 16 * wl.KIB, 64 * wl.MIB, 1.0, 64.0, False, "f32", 12000)
    w.W = [np.abs(x) + np.float32(1e-3) for x in w.W]
    dyn = w.dyn.copy()
    dyn[17, 3, 0], dyn[211, 0, 1], dyn[100, 2, 2] = np.inf, np.inf, np.nan
    scores, idx, best = Scorer(w).run(dyn=dyn)
    m = oracle_model(w)
    ref = orc.score(m, dyn, w.scal, w.part, w.cred)
    inf, nan = np.zeros(S, bool), np.zeros(S, bool)
    inf[[17, 211]], nan[100] = True, True
    assert np.isposinf(ref[inf]).all() and np.isnan(ref[nan]).all()
    assert np.isposinf(scores[inf]).all() and np.isnan(scores[nan]).all()
    assert (idx[inf] == 0).all() and idx[100] == -1
    rest = ~(inf | nan)
    assert np.linalg.norm(scores[rest] - ref[rest]) <= 1e-6 * np.linalg.norm(ref[rest])

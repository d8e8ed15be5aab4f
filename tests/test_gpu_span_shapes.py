"""Candidate counts that are no multiple of 256: the first hidden GEMM's row tiles span scenarios (csrc/gemm_span.hip).
The smallest count it takes (eight scenarios per tile), counts at every remainder modulo four, one below and above a
tile, two slabs per tile, a ragged last tile, grids per scenario; each against the fp64 oracle."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2112_13509_amd import workloads as wl
from gpu_helpers import Scorer, check_scores
from helpers import oracle_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,P,Q,hidden,own_grids", [
    (450, 37, 1, [256, 256], False),           # C = 37: eight scenarios in a tile, groups of four cross borders
    (451, 5, 8, [512, 256], False),            # C = 40: four adjacent rows share the partition value
    (300, 8, 8, [1024, 512, 256], True),       # C = 64: no group crosses a border
    (251, 11, 6, [256, 512], False),           # C = 66: rows 4j + 2 begin a scenario
    (200, 9, 11, [256, 256, 256], True),       # C = 99
    (65, 15, 17, [128, 1024, 256], False),     # C = 255, two slabs per tile
    (64, 16, 16, [128, 256], False),           # C = 256, two slabs per tile
    (66, 257, 1, [1024, 1024], False),         # C = 257
    (33, 25, 20, [192, 768, 256], True),       # C = 500, three slabs, three column tiles
    (9, 45, 41, [256, 256], False),            # C = 1845
])
def test_row_tiles_that_span_scenarios(S, P, Q, hidden, own_grids):
    w = wl.make_scoring("span-shapes", S, 16, hidden, P, Q, 16 * wl.KIB, 64 * wl.MIB, 1.0, 64.0, False, "bf16", 7000 + S)
    part = cred = None
    if own_grids:
        rng = np.random.default_rng(S)
        part = (w.part[None] * np.exp2(rng.uniform(-1, 1, (S, 1)))).astype(np.float32)
        cred = (w.cred[None] * rng.uniform(1, 1.25, (S, 1))).astype(np.float32)
    scores, idx, best = Scorer(w).run(part=part, cred=cred)
    ref = orc.score(oracle_model(w), w.dyn, w.scal, w.part if part is None else part, w.cred if cred is None else cred)
    err, checked = check_scores("bf16", scores, idx, ref)
    print("S=%d C=%d hidden=%s rel err %.3g, choice checked on %.0f%%" % (S, w.C, hidden, err, 100 * checked))
    assert np.array_equal(idx, np.argmax(scores, axis=1)) and np.array_equal(best, scores[np.arange(S), idx])

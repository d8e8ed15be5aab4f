"""Hidden products whose last (or only) round of 256 x 256 tiles goes in halves or quarters of tiles (gemm_big.hip, gemm_span.hip): as the
only item of a work-group and behind whole tiles, with parts that lie past the last row, generated and stored operands, both
epilogues; each against the fp64 oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2112_13509_amd import binding as ab
from paper_2112_13509_amd import workloads as wl
from gpu_helpers import Scorer, check_scores
from helpers import oracle_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,P,Q,hidden,own_grids,want", [
    # tiles of an XCD (32 work-groups each): the largest number decides the parts; want: of each hidden product, 0 on generic tiles
    (3, 16, 16, [512, 1024], False, [4]),                # 4 (or none): quarters, nothing but parts, fused output unit
    (13, 32, 8, [128, 1024], False, [4]),                # 8, two slabs a part
    (24, 16, 17, [1024, 1024], False, [2]),              # 16: halves, rows span scenarios, credit runs of odd length
    (20, 16, 16, [512, 1024, 256, 512], True, [2, 0, 0]),    # 12: halves, generic tiles behind them
    (44, 10, 10, [512, 512, 512, 64], True, [4, 4, 0]),  # 6: quarters of a generated and of a stored operand, both stored; last row tile of 48 rows
    (11, 16, 32, [512, 768, 768], False, [2, 2]),        # 9: halves, three column tiles; two scenarios of tiles
    (65, 16, 16, [256, 1024, 1024], False, [4, 4]),      # 36 and 32: quarters behind a whole tile on one XCD, none on the others
    (75, 16, 16, [128, 1024, 256], True, [4, 2]),        # 40 and 36: quarters behind a whole tile of two slabs; 10 and 9: halves of a stored operand
    (90, 16, 15, [256, 1024, 1024], False, [2, 2]),      # 44 and 40: halves behind a whole tile, rows span scenarios
    (90, 16, 16, [256, 1024, 1024], True, [2, 2]),       # 48 and 44: halves behind a whole tile
    (300, 16, 16, [256, 256, 64, 256], False, [4, 0, 4]),    # 38 and 37 of one column tile; K = 64 of a stored operand, one slab a part
    (70, 15, 17, [256, 1024, 1024], False, [4, 4]),      # last row tile of 186 rows: a quarter of it past the end
    (41, 10, 10, [512, 1024, 1024], True, [2, 2]),       # last row tile of four rows: a half of it past the end
    (41, 10, 10, [512, 512], True, [4]),                 # ... three quarters past the end
    (47, 37, 1, [512, 512], False, [4]),                 # eight scenarios a tile, groups of rows that cross borders
])
def test_last_round_in_parts(S, P, Q, hidden, own_grids, want):
    w = wl.make_scoring("parts", S, 16, hidden, P, Q, 16 * wl.KIB, 64 * wl.MIB, 1.0, 64.0, False, "bf16", 400 + S)
    f = ab.load()._ZN2ab22scoring_parts_of_tilesEPK13ab_model_descliii
    f.restype, f.argtypes = C.c_int, (C.c_void_p, C.c_int64, C.c_int32, C.c_int, C.c_int)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert [f(C.byref(ab.desc_from_workload(w)), S, w.C, k, cus) for k in range(1, len(hidden))] == want
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

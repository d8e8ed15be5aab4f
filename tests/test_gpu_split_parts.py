"""fp32 products whose weights lie in their parts (csrc/split_parts.hpp): each room of the workspace that holds them (the candidate
table's, the candidate rows', the second pass's) and none, one layer's weights and three, column tiles of 64, 128 and 256 in one group and in several,
two slabs and many, and the openings that lay them out.  Scores and the chosen candidate's vector against the fp64 oracle."""
import ctypes as C

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2112_13509_amd import binding as ab
from paper_2112_13509_amd import workloads as wl
from gpu_helpers import Scorer
from helpers import oracle_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,L,P,Q,hidden,own_grids,want", [
    (97, 16, 16, 17, [64, 64], False, [64]),                   # candidate table's room, joined opening; rows 16 short of a tile
    (2100, 30, 4, 3, [64, 192], True, [64]),                   # second pass's room, three column tiles
    (300, 350, 13, 7, [128, 128], False, [128]),               # candidate rows' room, opening without the product
    (520, 5, 4, 25, [256, 256], True, [128]),                  # second pass's room, two groups of one tile
    (260, 9, 20, 20, [256, 256, 256, 256, 256], False, [128, 128, 128, 0]),     # three layers at most: the fourth splits in its work-groups
    (96, 9, 16, 16, [256, 256], True, [0]),                    # no room
    (64, 9, 16, 24, [256, 256], True, [128]),                  # ... and just enough
    (600, 6, 16, 15, [256, 256], False, [256]),                # one group, one tile of 256; no whole row tile at the end
    (400, 6, 33, 16, [256, 512], False, [256]),                # two groups
    (130, 6, 36, 32, [320, 768], False, [256]),                # just enough room, three groups
    (300, 6, 32, 32, [256, 512], False, [256]),                # one group, two tiles
    (1100, 6, 16, 8, [128, 256], False, [128]),                # short sums: tiles of 128, two in a group
    (3600, 3, 20, 15, [64, 256], True, [128]),                 # second pass's room and two chunks: the first one's choice must leave it alone
])
def test_split_weights(S, L, P, Q, hidden, own_grids, want):
    w = wl.make_scoring("split-parts", S, L, hidden, P, Q, 16 * wl.KIB, 64 * wl.MIB, 1.0, 64.0, False, "f32", 21000 + S)
    f = ab.load()._ZN2ab18scoring_parts_tileEPK13ab_model_descliii
    f.restype, f.argtypes = C.c_int, (C.c_void_p, C.c_int64, C.c_int32, C.c_int, C.c_int)
    assert [f(C.byref(ab.desc_from_workload(w)), S, w.C, int(own_grids), k) for k in range(1, len(hidden))] == want
    part = cred = None
    if own_grids:
        rng = np.random.default_rng(S)
        part = (w.part[None] * np.exp2(rng.uniform(-1, 1, (S, 1)))).astype(np.float32)
        cred = (w.cred[None] * rng.uniform(1, 1.25, (S, 1))).astype(np.float32)
    scores, idx, best, v = Scorer(w).run(part=part, cred=cred, want_v=True)
    ref = orc.score(oracle_model(w), w.dyn, w.scal, w.part if part is None else part, w.cred if cred is None else cred)
    # as for the weights that each work-group splits: fp32 sums of up to a thousand terms are off by 2 to 5e-7, and by 2e-6 without one
    # of the three smallest partial products; a slab, part or tile in a wrong place is off by far more
    assert np.linalg.norm(scores - ref) <= 1e-6 * np.linalg.norm(ref)
    assert np.array_equal(idx, np.argmax(scores, axis=1)) and np.array_equal(best, scores[np.arange(S), idx])
    # one output: the vector is that candidate's score, computed by other kernels
    assert np.linalg.norm(v[:, 0] - best) <= 2e-6 * np.linalg.norm(best)

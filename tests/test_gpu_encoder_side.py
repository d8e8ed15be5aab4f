"""The scalars' columns and the layer-1 preparation in the encoders' launch, and the cases that keep launches of their own for them (a
large candidate table, statistics off 16 bytes); each against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2112_13509_amd import workloads as wl
from gpu_helpers import DEV, Scorer, check_scores
from helpers import oracle_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["mlp", "lstm"])
@pytest.mark.parametrize("S,hidden,P,Q,shift,own_grids", [
    (1, [64, 64], 3, 5, 0, False), (29, [128], 16, 8, 0, False),
    (3, [512], 40, 32, 0, False),                # 1280 candidates x 512 units: launches of their own
    (3, [512], 40, 32, 0, True),                 # ... no table with a grid per scenario
    (70, [256, 256], 16, 16, 1, True),           # statistics on 4 bytes
    (531, [64, 128], 5, 4, 0, False)])           # more scenarios than work-groups of the per-tensor encoder
def test_work_beside_the_encoders(kind, S, hidden, P, Q, shift, own_grids):
    make, sizes = (wl.make_lstm_encoder, {}) if kind == "lstm" else (wl.make_tensor_encoder, {"te_hidden": [128, 128]})
    w = make("side", S, hidden, P=P, Q=Q, dtype="bf16", seed=31 + S, n_blocks=1, per_block=9, extra=2, **sizes)
    part = cred = None
    if own_grids:
        rng = np.random.default_rng(S)
        part = (w.part[None] * np.exp2(rng.uniform(-1, 1, (S, 1)))).astype(np.float32)
        cred = (w.cred[None] * rng.uniform(1, 1.25, (S, 1))).astype(np.float32)
    flat = torch.zeros(w.dyn.size + shift, device=DEV)
    dyn = flat[shift:].view(w.dyn.shape)
    dyn.copy_(torch.from_numpy(w.dyn))
    scores, idx, best = Scorer(w).run(dyn=dyn, part=part, cred=cred)
    ref = orc.score(oracle_model(w), w.dyn, w.scal, w.part if part is None else part, w.cred if cred is None else cred)
    err, checked = check_scores("bf16", scores, idx, ref)
    print("%s S=%d C=%d hidden=%s rel err %.3g, choice checked on %.0f%%" % (kind, S, w.C, hidden, err, 100 * checked))
    assert np.array_equal(idx, np.argmax(scores, axis=1)) and np.array_equal(best, scores[np.arange(S), idx])

"""The online update's row-block form and its border to the layer-by-layer form, at the sizes where either can go wrong:
fewer and more rows than a block of 16 or 32, batches around the padding to 64, layers of one to sixteen 64-column slices
(one to eight wavefronts a slice, several passes), several outputs, every first trainable layer, and networks just too
wide or too heavy for the row-block form.  One step from a fresh state against the fp64 oracle, with the bounds of
test_gpu_update.gradient_bounds."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2112_13509_amd import binding as ab
from paper_2112_13509_amd import workloads as wl
from helpers import oracle_model, tensor_error, frob_error
from test_gpu_update import DEV, TOL, TOL_MATCHED, GpuTrainer, gradient_bounds

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, layers, hidden, rows, workers, first trainable layer
    ("f32", 3, (64,), 1, 0, 0), ("bf16", 3, (64,), 1, 0, 0),
    ("f32", 16, (128, 192), 15, 2, 0), ("bf16", 16, (128, 192), 17, 2, 0),
    ("f32", 21, (320, 64), 63, 0, 1), ("bf16", 21, (320, 64), 65, 0, 1),
    ("f32", 20, (256, 320), 129, 16, 0), ("bf16", 43, (576, 384), 129, 16, 0),
    ("bf16", 40, (1024, 512), 300, 0, 0), ("f32", 5, (640, 128), 300, 4, 2),
    ("bf16", 20, (512, 256, 192), 4097, 0, 1), ("f32", 6, (128, 64), 4097, 0, 0),
    ("bf16", 20, (256, 256), 513, 8, 2),
    # layer-by-layer form: a layer beyond 1024 columns, weights beyond 3.5 MB, fp32 activations beyond the LDS
    ("bf16", 8, (1088, 64), 130, 0, 0), ("bf16", 30, (1024, 1024, 1024), 100, 2, 1), ("f32", 4, (1024, 512), 70, 0, 0),
]


@pytest.mark.parametrize("dtype,L,hidden,B,n,first", CASES)
def test_step(dtype, L, hidden, B, n, first):
    u = wl.make_update("rows", N=max(B, 64), batch=B, L=L, hidden=hidden, dtype=dtype, seed=B + L, P=8, Q=8, n_workers=n,
                       loss_kind="l2norm" if n == 16 else "mse")
    tr, rows = GpuTrainer(u, B), np.arange(B)
    st = orc.TrainState.fresh(u.W, u.b)
    fw = [wl.bf16_round(w.astype(np.float32)).astype(np.float64) for w in st.W] if dtype == "bf16" else None
    tr.load_state(st)
    before = st.copy()
    p = tr.params
    idx = torch.from_numpy(rows).to(DEV)
    x, y = tr.x[idx].contiguous(), tr.y[idx].contiguous()
    kept = [t.clone() for t in p.W_master[:first] + p.b[:first]]
    if first:
        ab.ab_online_update_tail(tr.desc, p, x, y, first, loss_out=tr.loss, workspace=tr.ws)
    else:
        ab.ab_online_update(tr.desc, p, x, y, loss_out=tr.loss, workspace=tr.ws)
    gl = tr.loss_value()
    ref = orc.update(oracle_model(u), st, u.x_raw[rows], u.target[rows], forward_weights=fw, first_trainable=first)
    assert abs(gl - ref["loss"]) <= TOL[dtype] * abs(ref["loss"])
    bounds, refq = gradient_bounds(u, before, rows, ref, 1e-3, fw, first)
    for a, b in zip(kept, p.W_master[:first] + p.b[:first]):
        assert torch.equal(a, b)
    for k in range(first, len(hidden) + 1):
        gW, gb = (t.cpu().numpy().astype(np.float64) / 0.1 for t in (p.mW[k], p.mb[k]))     # m' = 0.1 g from a fresh state
        assert tensor_error(gW, ref["gW"][k]) <= bounds[k][0] and tensor_error(gb, ref["gb"][k]) <= bounds[k][1], k
        assert frob_error(gW, ref["gW"][k]) <= bounds[k][2] and frob_error(gb, ref["gb"][k]) <= bounds[k][3], k
        if refq is not None:
            for g, r, alone in ((gW, refq["gW"][k], bounds[k][0]), (gb, refq["gb"][k], bounds[k][1])):
                assert tensor_error(g, r) <= max(TOL_MATCHED, 0.4 * alone), k
        assert torch.equal(p.W[k], p.W_master[k].to(p.W[k].dtype))
    assert int(p.step.item()) == 1

"""The training step's fused backward kernels (input, weight and bias gradients
of a layer from one reading) against the FP64 reference with the GPU's BF16
roundings applied where it rounds: output gradient and hidden gradients.

What is left is FP32 accumulation (about 1e-6 of a value) and the BF16
roundings that it turns: a fraction of about 1e-6 / 2^-8 = 3e-4 of the entries
moves by 2^-8, 7e-5 relative L2 for each of six rounded tensors.  1e-3 is held;
a border row or column of a tile left out moves the sums by more than 2e-2."""
import numpy as np
import pytest

from oracle import cnn as ref
from test_gpu_cnn import _batch, _rel_l2, _setup

pytestmark = pytest.mark.gpu


# the narrowest tile (half a column chunk); three chunks, the last half empty;
# one chunk, several rows to a workgroup (640 workgroups of 4 rows would exceed
# the cap of 512)
@pytest.mark.parametrize("shape", [(1, 32, 32), (2, 32, 160), (40, 64, 64)])
def test_step_gradient_with_the_gpus_roundings(shape):
    import torch
    prop, wr, br, g, dev = _setup(21)
    x, mask, logq = _batch(g, *shape)
    T = lambda a: torch.from_numpy(a).to(dev)   # noqa: E731
    _, grad = prop.train_step(T(x), T(mask), T(logq), lr=1e-3, lam=0.1, want_grad=True)
    gr = grad.cpu().numpy().astype(np.float64)
    acts = ref.forward(x, wr, br, round_acts=True)
    _, dout = ref.loss(acts[-1], mask.astype(np.float64), logq.astype(np.float64), lam=0.1)
    dy, o, want = ref.bf16_round(dout), gr.size, []
    for l in (3, 2, 1, 0):
        xin = ref.bf16_round(acts[l])
        dw, db, dx = ref.conv3x3_backward(xin, wr[l], dy, need_dx=l > 0)
        want.insert(0, (dw, db))
        if l > 0:
            dy = ref.bf16_round(np.where(xin > 0, dx, 0.0))
    o = 0
    for l, (dw, db) in enumerate(want):
        ew = _rel_l2(gr[o:o + dw.size], dw)
        eb = _rel_l2(gr[o + dw.size:o + dw.size + db.size], db)
        print(f"layer {l} {shape}: grad rel L2 w {ew:.2e} b {eb:.2e}")
        assert ew <= 1e-3 and eb <= 1e-3
        o += dw.size + db.size

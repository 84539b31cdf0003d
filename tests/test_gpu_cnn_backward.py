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


@pytest.mark.parametrize("shape", [(1, 32, 32), (3, 32, 96), (2, 128, 64)])
def test_step_gradient_is_the_layers_in_a_row(shape):
    """The training step's fused passes against the same kernel one layer at a
    time (qsq_cnn_layer_backward: each held to the reference by itself), the
    gradient handed on masked and rounded by torch.  Both sum in one order, so
    only the loss gradient's exponential can differ, by a rounding: 1e-5, the
    bound of one layer's accumulation, is held."""
    import torch

    from paper_1609_00724_amd import learn
    prop, _, _, g, dev = _setup(31)
    x, mask, logq = (torch.from_numpy(a).to(dev) for a in _batch(g, *shape))
    lam, P = 0.1, mask.numel()
    acts = [x]
    for l in range(3):
        acts.append(learn.to_bf16_bits(learn.layer_forward(prop, l, acts[-1])))
    out = learn.layer_forward(prop, 3, acts[-1])
    sig = 1 / (1 + torch.exp(-out[..., 0]))
    dq = torch.where(torch.isfinite(logq), out[..., 1] - logq, torch.zeros_like(logq))
    dy = torch.stack([(sig - mask).double() / P, 2.0 * float(np.float32(lam)) * dq.double() / P], -1).float()
    want = []
    for l in (3, 2, 1, 0):
        dw, db, dx = learn.layer_backward(prop, l, acts[l], learn.to_bf16_bits(dy.contiguous()))
        want = [dw, db, *want]
        if l > 0:
            dy = torch.where(learn.from_bf16_bits(acts[l]) > 0, dx, torch.zeros_like(dx))
    _, grad = prop.train_step(x, mask, logq, lr=1e-3, lam=lam, want_grad=True)
    torch.cuda.synchronize()
    o = 0
    for k, w in enumerate(want):
        e = _rel_l2(grad[o:o + w.numel()].double().cpu().numpy(), w.double().cpu().numpy())
        print(f"layer {k // 2} {'b' if k % 2 else 'w'} {shape}: rel L2 {e:.2e}")
        assert e <= 1e-5
        o += w.numel()

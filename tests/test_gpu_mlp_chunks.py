"""The network's backward pass at the edges of its tiles (16 samples), chunks
(64), partial sums (16 threads, 4 partials each) and grid (512 workgroups),
against the FP64 oracle; weights at and off a 16-byte boundary give the same bits.

Bars as in the other tests of these kernels: every product runs on fp16
operands (relative rounding 5e-4), so the gradient is held to a relative L2
error of 1e-2 and the loss to 1e-3."""
import ctypes as C

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


def case(B, seed):
    rng = np.random.default_rng(seed)
    w = (rng.standard_normal(O.MLP_NPARAM) * 0.3).astype(np.float16)
    x = np.zeros((B, 32), dtype=np.float16)
    x[:, :27] = rng.uniform(-1, 1, (B, 27))
    return w, x, rng.uniform(-1, 1, (B, 4)).astype(np.float32)


def backward(w, x, t, shift=0):
    import torch

    from paper_2505_01126_amd import lbm

    B = len(x)
    buf = torch.zeros(len(w) + 8, dtype=torch.int16, device="cuda")
    buf[shift:shift + len(w)] = torch.tensor(w.view(np.int16), device="cuda")
    X, T = torch.tensor(x.view(np.int16), device="cuda"), torch.tensor(t, device="cuda")
    g = torch.full((len(w),), float("nan"), device="cuda")
    loss = torch.full((1,), float("nan"), device="cuda")
    y = torch.full((B, 4), float("nan"), device="cuda")
    work = torch.empty(lbm.lbm_mlp_work_bytes(B), dtype=torch.uint8, device="cuda")
    p = lambda a, o=0: C.c_void_p(a.data_ptr() + o)
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    lbm.lbm_mlp_backward(p(buf, 2 * shift), p(X), p(T), B, p(g), p(loss), p(work), work.numel(), st)
    lbm.lbm_mlp_forward(p(buf, 2 * shift), p(X), B, p(y), st)
    return g.cpu().numpy(), float(loss), y.cpu().numpy()


@pytest.mark.parametrize("B", [1, 15, 16, 17, 63, 64, 65, 1023, 1025, 4097, 32769])
def test_backward_at_the_edges(B):
    w, x, t = case(B, B)
    g, loss, y = backward(w, x, t)
    lo, go = O.mlp_loss_grad(w.astype(np.float64), x[:, :27].astype(np.float64), t.astype(np.float64))
    assert np.linalg.norm(g - go) < 1e-2 * np.linalg.norm(go)
    assert loss == pytest.approx(lo, rel=1e-3)
    yo = O.mlp_forward(w.astype(np.float64), x[:, :27].astype(np.float64))
    assert np.abs(y - yo).max() < 2e-3 * np.abs(yo).max()


@pytest.mark.parametrize("shift", [1, 4, 7])
def test_weights_off_a_16_byte_boundary(shift):
    w, x, t = case(200, 3)
    a, b = backward(w, x, t), backward(w, x, t, shift)
    assert np.array_equal(a[0], b[0]) and a[1] == b[1] and np.array_equal(a[2], b[2])

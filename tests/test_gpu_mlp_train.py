"""One training step of the column network at the batch sizes where its work is
split differently: 16 or 32 rows per workgroup (up to 4096, above), one to sixteen
batch slices of the weight gradients, slices of unequal length."""
import numpy as np
import pytest

from oracle import mlp_oracle as MO

pytestmark = pytest.mark.gpu

# The oracle below rounds the hidden activations to FP16 as the kernels do, so the
# two differ where FP32 rounding (1e-6 of a value) moves an activation across an FP16
# rounding boundary (2^-10 apart): a fraction f = 1e-6 / 2^-10 to 1e-2 of them, each by
# 2^-10.  In the norm that is sqrt(f) 2^-10 <= 1e-4; doubled for the layers.
TOL = 2e-4


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("B", [64, 192, 1984, 4096, 4160, 8512])
def test_train_step_over_batch_sizes(B):
    import torch
    from paper_2504_08157_amd import nhsem
    rng = np.random.default_rng(B)
    m = nhsem.ColumnMLP(max_batch=B)
    w = rng.normal(scale=0.08, size=m.nparam).astype(np.float32)
    m.nh_mlp_set_params(torch.from_numpy(w).cuda())
    x = rng.normal(size=(B, MO.IN)).astype(np.float16)
    t = rng.normal(scale=0.5, size=(B, MO.OUT)).astype(np.float32)

    def f16(a):
        return a.astype(np.float16).astype(np.float64)

    parts = MO.unflatten(w.astype(np.float64))
    for i in (0, 2, 4, 6):
        parts[i] = f16(parts[i])
    W1, b1, W2, b2, W3, b3, S = parts
    xo = x.astype(np.float64)
    z1 = xo @ W1.T + b1
    h1 = f16(MO.silu(z1))
    z2 = h1 @ W2.T + b2
    h2 = f16(MO.silu(z2))
    y = h2 @ W3.T + b3 + xo @ S.T
    go = MO.unflatten(MO.backward(MO.flatten(parts), (xo, z1, h1, z2, h2), MO.mse_grad(y, t.astype(np.float64))))

    # targets and dY at an address that is aligned to one float only
    buf = torch.empty(B * MO.OUT + 1, device="cuda")
    td = buf[1:].view(B, MO.OUT)
    td.copy_(torch.from_numpy(t))
    xd = torch.from_numpy(x).cuda()
    yd = m.nh_mlp_forward(xd)
    loss = torch.zeros(1, device="cuda")
    m.nh_mlp_train_step(xd, td, lr=1e-3, loss=loss)
    w1, g = m.nh_mlp_params()
    lo = MO.mse(y, t.astype(np.float64))
    assert abs(loss.item() - lo) <= TOL * lo, (loss.item(), lo)
    for i, (a, b) in enumerate(zip(MO.unflatten(g.cpu().numpy()), go)):
        assert _rel(a, b) <= TOL, (i, _rel(a, b))
    z = np.zeros(m.nparam)
    wa, _, _ = MO.adam(w.astype(np.float64), g.cpu().numpy().astype(np.float64), z, z, 1, 1e-3, 0.9, 0.999, 1e-8)
    assert np.linalg.norm(w1.cpu().numpy() - wa) <= 1e-5 * np.linalg.norm(wa - w)

    # forward and backward by themselves: the same gradient from the same numbers
    m.nh_mlp_set_params(torch.from_numpy(w).cuda())
    assert torch.equal(m.nh_mlp_forward(xd), yd)
    td.copy_(2.0 * (yd - td) * np.float32(1.0 / (B * MO.OUT)))
    m.nh_mlp_backward(xd, td)
    _, g2 = m.nh_mlp_params()
    assert _rel(g2.cpu().numpy(), g.cpu().numpy()) <= 1e-6
    # and again from the activations that the training step leaves behind
    m.nh_mlp_backward(xd, td)
    assert torch.equal(m.nh_mlp_params()[1], g2)

"""GPU tests of the network's fused launches (csrc/mlp.hip): products split over blocks whose last block goes on to
the elementwise work, the three products of a layer's backward pass in one launch; ragged, unaligned and one-row
sizes, K on either side of a staged step.

The reference rounds the operands of every product to BF16 as the kernels do and adds in FP64.  FP32 accumulation
of up to 4096 terms stays within 1e-5 of the largest value; a hidden value that lands on the other side of a BF16
rounding moves by 2^-8 of itself, which a few of the hundreds of values do: 2e-3 in the 2-norm of each gradient."""
import numpy as np
import pytest
import torch

from paper_1908_07392_amd import mhlp

pytestmark = pytest.mark.gpu


def _bf16(a):
    return torch.as_tensor(a, dtype=torch.float32).to(torch.bfloat16).double().numpy()


def _gelu(z):
    t = np.tanh(0.7978845608028654 * (z + 0.044715 * z ** 3))
    d = 0.7978845608028654 * (1 + 3 * 0.044715 * z * z)
    return 0.5 * z * (1 + t), 0.5 * (1 + t) + 0.5 * z * (1 - t * t) * d


@pytest.mark.parametrize("sizes,batch", [((64, 32, 32), 32), ((130, 33, 7), 1), ((1001, 65, 31), 129),
                                         ((4096, 256, 1024), 96), ((127, 300, 260), 200), ((3, 1, 1), 5)])
def test_step_against_fp64(sizes, batch):
    n_in, width, n_out = sizes
    rng = np.random.default_rng(n_in)
    net = mhlp.MLP(n_in, width, n_out, seed=1)
    w = [(rng.uniform(-1, 1, (b, a)) / np.sqrt(a), rng.uniform(-0.1, 0.1, b))
         for a, b in ((n_in, width), (width, width), (width, n_out))]
    w = [(a.astype(np.float32), b.astype(np.float32)) for a, b in w]
    p = torch.as_tensor(np.concatenate([np.concatenate([a.ravel(), b]) for a, b in w]), device="cuda:0")
    X, T = rng.standard_normal((batch, n_in)).astype(np.float32), rng.standard_normal((batch, n_out)).astype(np.float32)
    dev = [torch.as_tensor(v, device="cuda:0") for v in (X, T)]
    net.set_params(p)
    assert torch.equal(net.get_params(), p)
    acts, zs = [X], []
    for l, (a, b) in enumerate(w):
        z = _bf16(acts[-1]) @ _bf16(a).T + b
        zs.append(z)
        acts.append(_gelu(z)[0] if l < 2 else z)
    y = net.forward(dev[0]).cpu().numpy()
    assert np.linalg.norm(y - zs[2]) <= 2e-3 * np.linalg.norm(zs[2])
    loss, grad = net.loss_grad(*dev)
    assert abs(float(loss) - np.mean((zs[2] - T) ** 2)) <= 2e-3 * float(loss)
    d, parts = 2 * (zs[2] - T) / T.size, []
    for l in (2, 1, 0):
        parts = [_bf16(d).T @ _bf16(acts[l]), d.sum(axis=0)] + parts
        if l:
            d = (_bf16(d) @ _bf16(w[l][0])) * _gelu(zs[l - 1])[1]
    got, at = grad.cpu().numpy(), 0
    for want in parts:
        g = got[at:at + want.size].reshape(want.shape)
        at += want.size
        assert np.linalg.norm(g - want) <= 2e-3 * np.linalg.norm(want)
    for _ in range(3):  # the arrival counters are zero again after every launch; the sums have a fixed order
        loss2, grad2 = net.loss_grad(*dev)
        assert torch.equal(grad, grad2) and abs(float(loss2) - float(loss)) <= 1e-5 * float(loss)
    net.adam_step(lr=1e-3)  # the first step moves by lr where the gradient is well above eps
    g = torch.as_tensor(got, device="cuda:0")
    want = p - 1e-3 * g / (g.abs() + 1e-8)
    assert float((net.get_params() - want).abs().max()) <= 1e-6

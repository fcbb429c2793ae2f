"""Gradients of the indicator's network at the edges of its tiles of sixteen samples and beyond
the 256 blocks of a pass, against float64 (each entry a float32 sum of up to 5,000 terms of the
size of the largest: within 1e-5 of it); a training step is gradients and Adam, bit for bit."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import learned, ops
    rng = np.random.default_rng(8)
    feat = rng.normal(size=(6000, 4)).astype(np.float32)
    label = rng.normal(size=6000).astype(np.float32)
    return ops, ops.Context(0), learned.glorot_params(3), feat, label


def reference(params, feat, label):
    at = np.cumsum([0, 256, 64, 4096, 64, 4096, 64, 64, 1])
    p = torch.from_numpy(params.astype(np.float64)).requires_grad_(True)
    W1, b1, W2, b2, W3, b3, W4, b4 = (p[at[k]:at[k + 1]] for k in range(8))
    x = torch.from_numpy(feat).double()
    for W, b in ((W1, b1), (W2, b2), (W3, b3)):
        x = torch.tanh(x @ W.reshape(64, -1).T + b)
    y = x @ W4 + b4
    loss = ((y - torch.from_numpy(label).double()) ** 2).mean()
    (g,) = torch.autograd.grad(loss, p)
    return g.numpy(), float(loss.detach()), y.detach().numpy()


@pytest.mark.parametrize("batch", [1, 15, 16, 17, 333, 4096, 5000])
def test_pass_edges(env, batch):
    ops, ctx, params, feat, label = env
    print(f"[case] network pass, batch {batch}", flush=True)
    sel = np.random.default_rng(batch).choice(6000, batch, replace=False)
    ref, loss_ref, y_ref = reference(params, feat[sel], label[sel])
    ft, lt = torch.as_tensor(feat, device="cuda"), torch.as_tensor(label, device="cuda")
    st = torch.as_tensor(sel.astype(np.int32), device="cuda")
    net, other = (ops.Mlp(ctx, params, np.zeros(4), np.ones(4)) for _ in range(2))
    y = net.forward(ft[st.long()].contiguous()).cpu().numpy()
    assert np.abs(y - y_ref).max() < 1e-5
    g, loss = net.gradients(ft, lt, st)
    assert np.abs(g.cpu().numpy() - ref).max() < 1e-5 * np.abs(ref).max()
    assert abs(loss.item() - loss_ref) < 1e-5 * loss_ref
    net.adam_step(g)
    other.train_step(ft, lt, st)
    assert np.array_equal(net.params(), other.params())
    assert loss.item() == other.loss.item()

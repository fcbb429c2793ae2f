"""Gradients and training steps of the indicator's network on several streams, from the first call on,
and without a workspace.  Passes of different networks on one context are independent, as are gradient
calls of one network: each must give the bits it gives alone.  Without a workspace the blocks' sums are
added in no fixed order: float32 sums of up to 5,000 terms of the size of the largest, within 1e-5 of it."""

import numpy as np
import pytest
import torch

from test_gpu_mlp_tiles import reference

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import learned, ops
    rng = np.random.default_rng(8)
    feat = rng.normal(size=(6000, 4)).astype(np.float32)
    label = rng.normal(size=6000).astype(np.float32)
    ft, lt = torch.as_tensor(feat, device="cuda"), torch.as_tensor(label, device="cuda")
    sels = [torch.as_tensor(rng.choice(6000, 4096 - 100 * k, replace=False).astype(np.int32), device="cuda")
            for k in range(2)]
    nets = lambda ctx: [ops.Mlp(ctx, learned.glorot_params(3 + k), np.zeros(4), np.ones(4)) for k in range(2)]  # noqa: E731
    return ops, nets, feat, label, ft, lt, sels


def test_two_networks_on_two_streams(env):
    ops, nets, _, _, ft, lt, sels = env
    print("[case] two networks, two streams", flush=True)
    a, b = nets(ops.Context(0)), nets(ops.Context(0))  # b's networks share a context but no stream
    alone = [net.gradients(ft, lt, s)[0].clone() for net, s in zip(a, sels)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    got = [[], []]
    for _ in range(20):
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                got[k].append(b[k].gradients(ft, lt, sels[k])[0])
    torch.cuda.synchronize()
    for k in range(2):
        assert all(torch.equal(g, alone[k]) for g in got[k])
    for _ in range(20):
        for k in range(2):
            a[k].train_step(ft, lt, sels[k])
    for _ in range(20):
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                b[k].train_step(ft, lt, sels[k])
    torch.cuda.synchronize()
    for k in range(2):
        assert np.array_equal(a[k].params(), b[k].params())


def test_one_network_on_two_streams(env):
    ops, nets, _, _, ft, lt, sels = env
    print("[case] one network, two streams", flush=True)
    net = nets(ops.Context(0))[0]
    alone = [net.gradients(ft, lt, s)[0].clone() for s in sels]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    got = [[], []]
    for _ in range(20):
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                got[k].append(net.gradients(ft, lt, sels[k])[0])
    torch.cuda.synchronize()
    for k in range(2):
        assert all(torch.equal(g, alone[k]) for g in got[k])


def without_workspace(net, ft, lt, sel, g, loss):
    ctx, P = net.ctx, lambda t: t.data_ptr()
    ctx.bind_stream()
    ctx._check(ctx.lib.apx_mlp_gradients(ctx.h, net.h, P(ft), P(lt), P(sel), sel.numel(), P(g), P(loss)))


def test_first_call_of_a_context_is_captured(env):
    """Nothing is allocated by the library: the first gradient calls of a context are recorded into a
    graph, and every replay gives the eager result, with eager work in between."""
    ops, nets, _, _, ft, lt, sels = env
    print("[case] first call captured", flush=True)
    other = nets(ops.Context(0))[0]
    eager, loss = other.gradients(ft, lt, sels[0])
    eager, loss = eager.clone(), loss.clone()
    g2, l2 = torch.empty_like(eager), torch.empty_like(loss)
    without_workspace(other, ft, lt, sels[0], g2, l2)
    net = nets(ops.Context(0))[0]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g, l1 = net.gradients(ft, lt, sels[0])
        without_workspace(net, ft, lt, sels[0], g2, l2)
    for k in range(4):
        g.fill_(float(k))
        g2.fill_(float(k))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(g, eager) and torch.equal(l1, loss)
        assert (g2 - eager).abs().max() < 1e-5 * eager.abs().max()
        assert abs(l2.item() - loss.item()) < 1e-5 * loss.item()
        other.gradients(ft, lt, sels[1])


@pytest.mark.parametrize("batch", [1, 16, 17, 4096, 5000])
def test_without_workspace(env, batch):
    ops, nets, feat, label, ft, lt, _ = env
    print(f"[case] gradients without a workspace, batch {batch}", flush=True)
    net = nets(ops.Context(0))[0]
    sel = np.random.default_rng(batch).choice(6000, batch, replace=False)
    ref, loss_ref, _ = reference(net.params(), feat[sel], label[sel])
    g = torch.full((net.N_PARAMS,), 7.0, device="cuda")
    loss = torch.full((1,), 7.0, device="cuda")
    without_workspace(net, ft, lt, torch.as_tensor(sel.astype(np.int32), device="cuda"), g, loss)
    assert np.abs(g.cpu().numpy() - ref).max() < 1e-5 * np.abs(ref).max()
    assert abs(loss.item() - loss_ref) < 1e-5 * loss_ref

"""ACE scratch: after a call, no other of at most as many active atoms allocates, so that it can be
recorded into a graph: fewer atoms (whose tiles' pairs are shared among blocks), float32 after float64,
coefficient gradients after a call without, more atoms in the system.  Replays equal the eager call
(forces to 1e-12 eV/A: float64 sums of some 50 terms of O(1) in another order)."""

import pytest
import torch

import synth
from oracle import ace as oace
from synth import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first,then", [
    (("fp32", 18, 20000, False), ("fp32", 18, 16000, False)),
    (("fp32", 18, 20000, False), ("fp32", 18, 4096, False)),
    (("fp64", 18, 16000, False), ("fp32", 18, 16000, False)),
    (("fp64", 18, 3000, False), ("fp64", 18, 2500, True)),
    (("fp32", 13, 8500, False), ("fp32", 40, 8500, False)),
])
def test_later_calls_do_not_allocate(first, then):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import ops
    print(f"[case] scratch {first} then {then}", flush=True)
    prm = synth.ace_random(10, 4, oace.num_basis(10, 4), seed=3)

    def setup(ctx, model, precision, cells, n_act, dc):
        atoms = ops.device_atoms(configs.bulk(cells, seed=2, sigma=0.08))
        nl = ops.build_neighbors(ctx, atoms, 5.5)
        active = torch.arange(n_act, dtype=torch.int32, device="cuda")
        return lambda: ops.ace_energy_forces(ctx, atoms, nl, model, active, None, precision, want_dc=dc)

    keys = ("e_site", "dE_dc1", "dE_dc2")
    other = ops.Context(0)
    ref = setup(other, ops.AceModel(other, prm), *then)()
    ctx = ops.Context(0)
    model = ops.AceModel(ctx, prm)
    warm, call = setup(ctx, model, *first), setup(ctx, model, *then)
    warm()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call()
    for _ in range(3):
        for t in out.values():
            if torch.is_tensor(t):
                t.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        for k in keys:
            if ref.get(k) is not None:
                assert torch.equal(out[k], ref[k]), k
        assert (out["f"] - ref["f"]).abs().max().item() < 1e-12
        warm()
        torch.cuda.synchronize()

"""New coefficients set from another stream than the default one, on which evaluations are still queued:
those end with the coefficients they began with."""

import pytest
import torch

import synth
from oracle import ace as oace
from synth import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_queued_evaluations_keep_their_coefficients(precision):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import ops
    print(f"[case] coefficients set behind queued evaluations, {precision}", flush=True)
    ctx = ops.Context(0)
    s = configs.bulk(32, seed=2, sigma=0.08)
    atoms = ops.device_atoms(s)
    nl = ops.build_neighbors(ctx, atoms, 5.5)
    nb = oace.num_basis(10, 4)
    a, b = synth.ace_random(10, 4, nb, seed=3), synth.ace_random(10, 4, nb, seed=4)
    model = ops.AceModel(ctx, a)
    active = torch.arange(s.n, dtype=torch.int32, device="cuda")
    run = lambda: ops.ace_energy_forces(ctx, atoms, nl, model, active, None, precision)["e_site"]  # noqa: E731
    ref = run()
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    queued = [run() for _ in range(4)]
    with torch.cuda.stream(other):
        model.set_coeffs(b.c1, b.c2)
    torch.cuda.synchronize()
    assert all(torch.equal(e, ref) for e in queued)
    assert not torch.equal(run(), ref)

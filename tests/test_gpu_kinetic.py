"""Kinetic energy of the integrator's statistics where its blocks take one round of atoms, several, and
part of one: a sum of n terms of equal sign, within n unit roundoffs of the sum in numpy."""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 257, 262144, 262145, 600001])
def test_kinetic_energy(n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print(f"[case] {n} atoms", flush=True)
    rng = np.random.default_rng(n)
    from paper_2411_03002_amd import ops
    L = 9.0 * np.ceil(n ** (1.0 / 3.0)) + 20.0
    m = int(np.ceil(n ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*([9.0 * np.arange(m)] * 3), indexing="ij")).reshape(3, -1)[:, :n] + 5.0
    s = synth.System(g, np.zeros(3), np.full(3, L), (1, 1, 1))
    vel = torch.as_tensor(rng.normal(0.0, 3.0, (3, n)), device="cuda")
    ctx = ops.Context(0)
    atoms = ops.device_atoms(s)
    md = ops.MD(ctx, atoms, synth.eam_cu_like(), None, None, mode="eam")
    pos = atoms.pos.clone()
    f, w = md.init(pos)
    e_kin = md.step(pos, vel, f, w, 0)["e_kin"]
    want = 0.5 * 63.546 / 9648.5332 * float((vel.cpu().numpy() ** 2).sum())
    assert abs(e_kin - want) < n * 2.3e-16 * want + 4e-16 * want

"""Compaction around the largest count that one block scans (16,384) and at the edges of its threads:
the active list is the ascending list of the atoms whose mask is set, whatever the number of atoms."""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 16383, 16384, 16385, 20481])
def test_active_list(n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import ops
    print(f"[case] {n} atoms", flush=True)
    rng = np.random.default_rng(n)
    L = 8.0 * np.ceil(n ** (1.0 / 3.0)) + 16.0  # a thin gas: as many cells as atoms and more
    s = synth.System(rng.uniform(0.0, L, (3, n)), np.zeros(3), np.full(3, L), (1, 1, 1))
    ctx = ops.Context(0)
    atoms = ops.device_atoms(s)
    nl = ops.build_neighbors(ctx, atoms, 5.5)
    csp = rng.uniform(0.0, 5.0, n)
    prm = synth.PrecisionParams(2.5, 3.0, 1, 0.0, 0.0)
    got = ops.compute_precision(ctx, atoms, nl, prm, csp=torch.as_tensor(csp, device="cuda"))
    mask = got["mask"].cpu().numpy()
    assert np.array_equal(mask != 0, got["w"].cpu().numpy() > 0.0)
    assert np.array_equal(got["active"].cpu().numpy(), np.flatnonzero(mask))

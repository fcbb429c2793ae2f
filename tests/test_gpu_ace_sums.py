"""Rounding of the float32 product sums: one call over 37,044 atoms (a block sums all of a tile's label
pairs) against calls of 1,400 (eight blocks share them).  The atomic bases are the same bits, so that the
site energies differ by the rounding of the sums alone.  The bounds are sqrt(2) times the rounding that
compensated float32 sums over the pairs leave, emulated in numpy for environments of this kind (12,3:
4.6e-9 eV RMS; 6,4: 7.3e-9; 10,4: 8.0e-9; 12,4: 8.9e-9); one float32 accumulator over all pairs leaves 2 to 5 times
as much (2.1e-8, 3.0e-8, 1.8e-8, 1.9e-8)."""

import pytest
import torch

import synth
from oracle import ace as oace
from synth import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_max,l_max,seed,rounding", [(12, 3, 1, 4.6e-9), (6, 4, 1, 7.3e-9), (10, 4, 2, 8.0e-9),
                                                       (12, 4, 1, 8.9e-9)])
def test_rounding_of_the_sums(n_max, l_max, seed, rounding):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import ops
    print(f"[case] float32 sums n_max {n_max} l_max {l_max}", flush=True)
    ctx = ops.Context(0)
    s = configs.bulk(21, seed=3, sigma=0.08)
    atoms = ops.device_atoms(s)
    nl = ops.build_neighbors(ctx, atoms, 5.5)
    model = ops.AceModel(ctx, synth.ace_random(n_max, l_max, oace.num_basis(n_max, l_max), seed=seed))
    every = torch.arange(s.n, dtype=torch.int32, device="cuda")
    one = ops.ace_energy_forces(ctx, atoms, nl, model, every, None, "fp32")["e_site"]
    parts = sum(ops.ace_energy_forces(ctx, atoms, nl, model, p, None, "fp32")["e_site"] for p in every.split(1400))
    assert (one - parts).square().mean().sqrt().item() < 2.0 ** 0.5 * rounding

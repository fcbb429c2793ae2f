"""ACE at the edges of the product kernels' tiles and of their instantiations.

The kernels hold 64 (float32) or 16 (float64) atoms per tile and are instantiated for 8, 10 and
12 radial functions; a call with few tiles shares a tile's label pairs among blocks, one with
many finishes each tile in its block.  Site energies and forces of every combination against
the oracle (float64 within 1e-10 eV and eV/A; float32 within 1e-5, the rounding bound of the
float32 path: sums of O(1e4) products of O(1) values with unit roundoff 6e-8).
"""

import numpy as np
import pytest
import torch

import synth
from oracle import ace as oace
from oracle import geometry
from synth import configs

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-10, "fp32": 1e-5}


@pytest.fixture(scope="module")
def env():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import ops
    s = configs.slab100(4, 4, 5, seed=77, frozen_planes=0, sigma=0.08, velocities=False)
    ctx = ops.Context(0)
    atoms = ops.device_atoms(s)
    nl = ops.build_neighbors(ctx, atoms, 5.5)
    i, j = geometry.pairs_within(s.pos, s.lo, s.hi, s.periodic, 5.0)
    return ops, ctx, s, atoms, nl, i, j


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n_max,l_max,n_act", [
    (1, 3, 17), (2, 4, 63), (5, 4, 1), (7, 3, 64), (8, 4, 65), (9, 3, 16), (9, 4, 129), (10, 3, 15), (11, 3, 33),
    (11, 4, 32), (12, 3, 81), (12, 4, 320)])
def test_tile_edges(env, precision, n_max, l_max, n_act):
    ops, ctx, s, atoms, nl, i, j = env
    print(f"[case] n_max {n_max} l_max {l_max} n_act {n_act} {precision}", flush=True)
    prm = synth.ace_random(n_max, l_max, oace.num_basis(n_max, l_max), seed=5, anchored=n_max % 2 == 1)
    rng = np.random.default_rng(n_act)
    sites = np.sort(rng.choice(s.n, n_act, replace=False))
    w = rng.uniform(0.1, 1.0, s.n)
    model = ops.AceModel(ctx, prm)
    out = ops.ace_energy_forces(ctx, atoms, nl, model, torch.as_tensor(sites.astype(np.int32), device="cuda"),
                                torch.as_tensor(w, device="cuda"), precision)
    pt = torch.tensor(s.pos, dtype=torch.float64, requires_grad=True)
    e = oace.site_energies(pt, s.box, s.periodic, i, j, prm, s.n, sites)
    (g,) = torch.autograd.grad((torch.as_tensor(w) * e).sum(), pt)
    tol = TOL[precision]
    assert np.abs(out["e_site"].cpu().numpy() - e.detach().numpy()).max() < tol
    assert np.abs(out["f"].cpu().numpy() + g.numpy()).max() < tol


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_many_tiles_equal_few(env, precision):
    """33,000 atoms in one call (a block finishes its tile) against calls of at most 1,500 atoms
    (blocks share a tile's pairs): the same sums in another order."""
    ops, ctx = env[0], env[1]
    s = configs.bulk(21, seed=3, sigma=0.08)
    atoms = ops.device_atoms(s)
    nl = ops.build_neighbors(ctx, atoms, 5.5)
    prm = synth.ace_random(10, 4, oace.num_basis(10, 4), seed=5)
    model = ops.AceModel(ctx, prm)
    every = torch.arange(33000, dtype=torch.int32, device="cuda")
    one = ops.ace_energy_forces(ctx, atoms, nl, model, every, None, precision)
    e = torch.zeros_like(one["e_site"])
    f = torch.zeros_like(one["f"])
    for part in every.split(1500):
        o = ops.ace_energy_forces(ctx, atoms, nl, model, part, None, precision)
        e += o["e_site"]
        f += o["f"]
    tol = TOL[precision]
    assert (one["e_site"] - e).abs().max().item() < tol
    assert (one["f"] - f).abs().max().item() < tol


@pytest.mark.parametrize("n_max,l_max,n_act", [(1, 3, 1), (2, 4, 31), (8, 3, 32), (9, 4, 33), (11, 3, 65), (12, 4, 97)])
def test_gradient_edges(env, n_max, l_max, n_act):
    """Coefficient gradients at the edges of their chunks of 32 atoms and groups of 16 pairs:
    float64 within 1e-10, float32 within 1e-5 of the largest component."""
    ops, ctx, s, atoms, nl, i, j = env
    print(f"[case] gradient n_max {n_max} l_max {l_max} n_act {n_act}", flush=True)
    prm = synth.ace_random(n_max, l_max, oace.num_basis(n_max, l_max), seed=5)
    rng = np.random.default_rng(n_act)
    sites = np.sort(rng.choice(s.n, n_act, replace=False))
    w = rng.uniform(0.1, 1.0, s.n)
    model = ops.AceModel(ctx, prm)
    act, wt = torch.as_tensor(sites.astype(np.int32), device="cuda"), torch.as_tensor(w, device="cuda")
    o64 = ops.ace_energy_forces(ctx, atoms, nl, model, act, wt, "fp64", want_dc=True)
    o32 = ops.ace_energy_forces(ctx, atoms, nl, model, act, wt, "fp32", want_dc=True)
    plain = ops.ace_energy_forces(ctx, atoms, nl, model, act, wt, "fp64")
    c1 = torch.tensor(prm.c1, requires_grad=True)
    c2 = torch.tensor(prm.c2, requires_grad=True)
    e = oace.site_energies(torch.as_tensor(s.pos), s.box, s.periodic, i, j, prm, s.n, sites, c1, c2)
    for key, g in zip(("dE_dc1", "dE_dc2"), torch.autograd.grad((torch.as_tensor(w) * e).sum(), (c1, c2))):
        g = g.numpy()
        assert np.abs(o64[key].cpu().numpy() - g).max() < 1e-10, key
        assert np.abs(o32[key].cpu().numpy() - g).max() < 1e-5 * np.abs(g).max(), key
    assert (o64["e_site"] - plain["e_site"]).abs().max().item() < 1e-10
    assert (o64["f"] - plain["f"]).abs().max().item() < 1e-10


def test_gradient_of_many_chunks(env):
    """9,000 atoms (more chunks than blocks, each block adds to its own sum) against parts."""
    ops, ctx = env[0], env[1]
    s = configs.bulk(14, seed=4, sigma=0.08)
    atoms = ops.device_atoms(s)
    nl = ops.build_neighbors(ctx, atoms, 5.5)
    model = ops.AceModel(ctx, synth.ace_random(8, 3, oace.num_basis(8, 3), seed=5))
    every = torch.arange(9000, dtype=torch.int32, device="cuda")
    one = ops.ace_energy_forces(ctx, atoms, nl, model, every, None, "fp64", want_dc=True)
    for key in ("dE_dc1", "dE_dc2"):
        parts = sum(ops.ace_energy_forces(ctx, atoms, nl, model, p, None, "fp64", want_dc=True)[key]
                    for p in every.split(700))
        assert (one[key] - parts).abs().max().item() < 1e-12 * one[key].abs().max().item()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n_max,l_max,anchored", [(10, 4, True), (9, 4, False), (8, 3, True), (12, 3, False)])
def test_dense_rows(env, precision, n_max, l_max, anchored):
    """A crystal compressed by 15 % along each axis: more neighbours inside the cutoff than the atomic
    base takes at a time (48), and rows of more than 64.  The tolerances are scaled by the largest force
    over that of the crystal at rest (about 1 eV/A)."""
    ops, ctx = env[0], env[1]
    print(f"[case] dense rows n_max {n_max} l_max {l_max} {precision}", flush=True)
    s = configs.slab100(4, 4, 5, seed=78, frozen_planes=0, sigma=0.05, velocities=False)
    s = synth.System(s.pos * 0.85, s.lo * 0.85, s.hi * 0.85, s.periodic)
    atoms = ops.device_atoms(s)
    nl = ops.build_neighbors(ctx, atoms, 5.5, max_nb=128)
    i, j = geometry.pairs_within(s.pos, s.lo, s.hi, s.periodic, 5.0)
    assert np.bincount(i).max() > 64 and nl.needed > 64
    prm = synth.ace_random(n_max, l_max, oace.num_basis(n_max, l_max), seed=6, anchored=anchored)
    sites = np.arange(s.n)
    w = np.random.default_rng(3).uniform(0.1, 1.0, s.n)
    out = ops.ace_energy_forces(ctx, atoms, nl, ops.AceModel(ctx, prm),
                                torch.as_tensor(sites.astype(np.int32), device="cuda"),
                                torch.as_tensor(w, device="cuda"), precision)
    pt = torch.tensor(s.pos, dtype=torch.float64, requires_grad=True)
    e = oace.site_energies(pt, s.box, s.periodic, i, j, prm, s.n, sites)
    (g,) = torch.autograd.grad((torch.as_tensor(w) * e).sum(), pt)
    tol = TOL[precision] * max(1.0, float(g.abs().max()))
    assert np.abs(out["e_site"].cpu().numpy() - e.detach().numpy()).max() < tol
    assert np.abs(out["f"].cpu().numpy() + g.numpy()).max() < tol

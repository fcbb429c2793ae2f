"""Kernels that gather over neighbour rows, at the sizes where the number of waves per 64 atoms
changes, and at the edges of a group of 64.

A periodic block repeated along the axes is the same crystal: what an atom gets there (more atoms, so
fewer waves per group) is what it gets in the block alone, whose values the oracle's tests cover.  The
rows differ in order, so sums agree to their rounding: at most 80 terms of up to 10 in eV and eV/A with
unit roundoff 1.1e-16, below 1e-12; 1e-10 is the bound used with the oracle.  Centro-symmetry is exact
arithmetic in a fixed order: bit-equal to the same operations in torch.
"""

import numpy as np
import pytest
import torch

import synth
from synth import configs

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.fixture(scope="module")
def env():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import ops
    return ops, ops.Context(0)


def repeat(s, reps):
    box = s.hi - s.lo
    parts = [s.pos + (np.array([a, b, c]) * box)[:, None]
             for a in range(reps[0]) for b in range(reps[1]) for c in range(reps[2])]
    return synth.System(np.concatenate(parts, axis=1), s.lo, s.lo + box * np.array(reps), s.periodic)


def exact_csp(pos, box, nl, rc):
    """The 12 nearest by (distance, index), the 6 smallest pair sums in ascending order, in the
    operation order of the kernels."""
    def near(d):
        for k in range(3):
            h = 0.5 * box[k]
            d[k] = torch.where(d[k] >= h, d[k] - box[k], torch.where(d[k] < -h, d[k] + box[k], d[k]))
        return d

    def square(d):
        return d[0] * d[0] + d[1] * d[1] + d[2] * d[2]

    n, m = pos.shape[1], nl.max_nb
    out = torch.empty(n, dtype=torch.float64, device=pos.device)
    for a in range(0, n, 20000):
        b = min(n, a + 20000)
        live = torch.arange(m, device=pos.device)[:, None] < nl.count[None, a:b]
        j = torch.where(live, nl.idx[:, a:b], 0).long()
        d = near([pos[k][j] - pos[k, a:b] for k in range(3)])
        r2 = torch.where(live, square(d), torch.inf)
        r2 = torch.where(r2 < rc * rc, r2, torch.inf)
        key, order = torch.sort(r2, dim=0, stable=True)
        x = [t.gather(0, order[:12]) for t in d]
        v = torch.stack([square([t[p] + t[q] for t in x]) for p in range(12) for q in range(p + 1, 12)])
        v = torch.sort(v, dim=0).values
        c = v[0]
        for q in range(1, 6):
            c = c + v[q]
        out[a:b] = torch.where(key[11] < torch.inf, c, torch.inf)
    return out


@pytest.mark.parametrize("n", [2, 63, 64, 65, 863])
def test_groups(env, n):
    """Atoms cut out of a crystal, open on all sides: rows from 0 entries up, the last group ragged."""
    ops, ctx = env
    print(f"[case] groups {n}", flush=True)
    full = configs.bulk(6, seed=3, temperature=300.0)
    far = np.argsort(((full.pos - full.pos.mean(axis=1)[:, None]) ** 2).sum(axis=0), kind="stable")
    s = synth.System(full.pos[:, np.sort(far[:n])], full.lo - 20.0, full.hi + 20.0, (0, 0, 0))
    atoms = ops.device_atoms(s)
    nl = ops.build_neighbors(ctx, atoms, 5.5)
    from oracle import geometry, hybrid
    w = np.random.default_rng(n).uniform(0.0, 1.0, s.n)
    e = ops.eam_forces(ctx, atoms, nl, synth.eam_cu_like(), torch.as_tensor(w, device="cuda"))
    ref = hybrid.evaluate(s, synth.eam_cu_like(), None, w, geometry.neighbor_csr(s.pos, s.lo, s.hi, s.periodic, 5.5))
    assert np.abs(e["f"].cpu().numpy() - ref["f_eam"]).max() < TOL
    pos = torch.as_tensor(s.pos, device="cuda")
    pr = ops.compute_precision(ctx, atoms, nl, synth.precision_hyb1())
    assert torch.equal(pr["csp"], exact_csp(pos, s.hi - s.lo, nl, synth.precision_hyb1().r_cut))


@pytest.mark.parametrize("reps", [(2, 3, 1), (2, 2, 2), (3, 3, 3), (4, 4, 5)])
def test_repeated_block(env, reps):
    ops, ctx = env
    base = configs.bulk(10, seed=21, temperature=300.0, vacancies=11)
    big = repeat(base, reps)
    print(f"[case] block of {base.n} repeated {reps}: {big.n} atoms", flush=True)
    w = np.random.default_rng(1).uniform(0.0, 1.0, base.n)
    got = []
    for s in (base, big):
        atoms = ops.device_atoms(s)
        ws = torch.as_tensor(np.tile(w, s.n // base.n), device="cuda")
        one = {}
        for name, pot, rl, nb in (("closed", synth.eam_cu_like(), 5.5, 80), ("two", synth.eam2_fit300k(), 6.0, 96)):
            nl = ops.build_neighbors(ctx, atoms, rl, max_nb=nb)
            e = ops.eam_forces(ctx, atoms, nl, pot, ws)
            one.update({f"{name} {k}": e[k] for k in ("e_site", "rho", "f")})
            if name == "closed":
                pr = ops.compute_precision(ctx, atoms, nl, synth.precision_hyb1())
                pos = torch.as_tensor(s.pos, device="cuda")
                assert torch.equal(pr["csp"], exact_csp(pos, s.hi - s.lo, nl, synth.precision_hyb1().r_cut))
                one["features"] = ops.features(ctx, atoms, nl, e["rho"], e["rho"], e["f"])
        got.append(one)
    for k, small in got[0].items():
        large = got[1][k]
        copies = large.reshape(*large.shape[:-1], -1, base.n) if large.shape[-1] == big.n else \
            large.reshape(-1, base.n, large.shape[-1])
        ref = small.unsqueeze(-2) if large.shape[-1] == big.n else small.unsqueeze(0)
        # features are float32 values of the sums
        tol = 1e-5 if k == "features" else TOL
        assert (copies - ref).abs().max() < tol, k


@pytest.mark.parametrize("cells,reps", [(6, (1, 1, 1)), (10, (3, 3, 3))])
def test_ties(env, cells, reps):
    """A static crystal with vacancies: equal distances (to rounding) at the twelfth neighbour."""
    ops, ctx = env
    s = repeat(configs.bulk(cells, seed=4, vacancies=9), reps)
    print(f"[case] ties {s.n}", flush=True)
    atoms = ops.device_atoms(s)
    nl = ops.build_neighbors(ctx, atoms, 5.5)
    pr = ops.compute_precision(ctx, atoms, nl, synth.precision_hyb1())
    want = exact_csp(torch.as_tensor(s.pos, device="cuda"), s.hi - s.lo, nl, synth.precision_hyb1().r_cut)
    assert torch.equal(pr["csp"], want)

"""What the library is measured on: the work a simulation with the adaptive-precision
EAM-ACE potential has it do, through the public calls of ``paper_2411_03002_amd``.

Kinds of case (field ``kind``):

* ``eval``   one static evaluation in float64 of a small cell, as a relaxation or a parity
  check makes it: neighbour list, weights, EAM, ACE on the detected atoms, blend.
* ``eam``    neighbour list and classical EAM (closed form or the EAM2 copper potential).
* ``weights``  centro-symmetry, switching and spreading on a list that is in hand.
* ``ace``    float64 ACE energies and forces of the detected atoms.
* ``grad``   ACE energy and its position gradient under autograd.
* ``fit``    one coefficient-fitting step: ACE energy, gradients of both coefficient
  vectors, update.
* ``train``  gradients of the learned indicator's network on one mini-batch.
* ``indicator``  the learned indicator deployed: features, bfloat16 inference, weight.
* ``md``     a segment of velocity-Verlet steps from a restart point, the time-averaged
  weights and the local thermostat as options.

The float32 evaluation of the autograd kinds stands in a float32 program: its leaves
(positions, coefficients) are float32 and so are the energy and the gradients it takes.
"""

import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2411_03002_amd import autograd, learned, ops

A_LAT = 3.615       # FCC lattice constant, Angstrom
MASS = 63.546       # amu
KB = 8.617333262e-5  # eV/K
CONV = 9648.5332    # 1 eV/amu in A^2/ps^2
RC, TAPER = 5.0, 0.5
SIGMA_300 = 0.08    # thermal displacement per component near 300 K, Angstrom


# ------------------------------------------------------------------------ parameters
def closed(alpha, beta, A):
    return SimpleNamespace(A=A, alpha=alpha, beta=beta, r0=A_LAT / math.sqrt(2.0), rc=RC, h=TAPER)


FAST = closed(4.3, 1.8, 0.1464436514321396)      # the fast potential
ANCHOR = closed(4.4, 1.75, 0.14169266975963063)  # the classical part of the precise one
# the EAM2 copper potential refit at 300 K (Appendix E, Table III)
EAM2 = SimpleNamespace(E1=2.01486e+02, E2=6.44057e-03, delta=2.18016e-02, alpha1=2.96972e+00, alpha2=1.55510e+00,
                       r01=8.36347e-01, r02=4.46690e+00, S=(4.0, 40.0, 1150.0), rs=(2.24, 1.80, 1.20),
                       a=3.80541e+00, beta1=1.66589e-01, beta2=5.35661e+02, r03=-2.19834e+00, r04=-2.61984e+02,
                       xi0=-2.30089e+00, xi2=1.39912e+00, q=(-1.29894e+00, -8.99672e-01, 1.79940e+00, 2.99944e+00),
                       Q1=3.99178e-01, Q2=3.00455e-01, f0=-1.50036e-01, rc=5.50679e+00, h=5.00370e-01)
PLAIN = SimpleNamespace(csp_lo=0.2, csp_hi=0.5, switch_kind=0, r_lo=0.0, r_hi=0.0, n_nn=12, n_buffer=0, r_cut=RC)
HYB1 = SimpleNamespace(csp_lo=2.5, csp_hi=3.0, switch_kind=1, r_lo=4.0, r_hi=12.0, n_nn=12, n_buffer=0, r_cut=RC)


@functools.lru_cache(maxsize=None)
def triples(n_max, l_max):
    """The labels (n, l) of every third-order basis function, in the basis order."""
    lab = [(n, l) for n in range(n_max) for l in range(l_max + 1)]
    out = []
    for p1 in range(len(lab)):
        for p2 in range(p1, len(lab)):
            for p3 in range(p2, len(lab)):
                a, b, c = lab[p1][1], lab[p2][1], lab[p3][1]
                if (a + b + c) % 2 == 0 and abs(a - b) <= c <= a + b:
                    out.append((lab[p1], lab[p2], lab[p3]))
    return out


def ace_params(n_max, l_max, anchored, seed):
    """Random ACE of the given size; the radial mixing and the coefficients from ``seed``."""
    rng = np.random.default_rng(seed)
    nb = ops.num_basis(n_max, l_max)
    W = rng.normal(0.0, 1.0 / math.sqrt(n_max), size=(l_max + 1, n_max, n_max))
    c1, c2 = rng.normal(0.0, 0.01, size=nb), rng.normal(0.0, 0.01, size=nb)
    return SimpleNamespace(n_max=n_max, l_max=l_max, W=W, c1=c1, c2=c2, rc=RC, h=TAPER, s_a=6.0, eps=0.1,
                           anchor=ANCHOR if anchored else None)


# ------------------------------------------------------------------------- geometries
def phonons(case, sites, g):
    """Thermal displacements of the sites: white noise on the grid of half cells, weighted by
    1/omega(k) of a nearest-neighbour lattice, so that neighbours move together as they do in
    a harmonic crystal (independent displacements would set off the centro-symmetry criterion
    almost everywhere at 300 K), scaled to the case's sigma per component."""
    dev = sites.device
    N = [2 * case["nx"], 2 * case["ny"], 2 * case["nz"]]
    om2 = torch.full((N[2], N[1], N[0]), 1e-3, dtype=torch.float64, device=dev)
    for axis, m in zip((2, 1, 0), N):
        shape = [1, 1, 1]
        shape[axis] = m
        om2 = om2 + torch.sin(math.pi * torch.arange(m, device=dev, dtype=torch.float64) / m).reshape(shape) ** 2
    flt = om2.rsqrt()
    flt[0, 0, 0] = 0.0
    at = torch.round(2.0 * sites).to(torch.int64)
    u = []
    for _ in range(3):
        white = torch.randn(om2.shape, generator=g, device=dev, dtype=torch.float64)
        v = torch.fft.ifftn(torch.fft.fftn(white) * flt).real[at[2], at[1], at[0]]
        u.append(v * (case["sigma"] / v.std()))
    return torch.stack(u)


def crystal(case, seed, device="cuda"):
    """An FCC block of the case's cells with its defects and thermal displacements:
    positions [3, n], box, periodicity, frozen mask and Maxwell velocities."""
    g = torch.Generator(device=device).manual_seed(1000003 * int(seed) + 17)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    ix = torch.arange(nx, device=device, dtype=torch.float64)
    iy = torch.arange(ny, device=device, dtype=torch.float64)
    iz = torch.arange(nz, device=device, dtype=torch.float64)
    zz, yy, xx = torch.meshgrid(iz, iy, ix, indexing="ij")
    cells = torch.stack([xx.reshape(-1), yy.reshape(-1), zz.reshape(-1)])
    basis = torch.tensor([[0.0, 0.0, 0.0], [0.5, 0.5, 0.0], [0.5, 0.0, 0.5], [0.0, 0.5, 0.5]], device=device,
                         dtype=torch.float64)
    sites = (cells[:, :, None] + basis.T[:, None, :]).reshape(3, -1)
    pos = torch.cat([sites * A_LAT, phonons(case, sites, g)])  # rows 3..5: displacements
    slab = case["shape"] == "slab"
    L = [nx * A_LAT, ny * A_LAT, nz * A_LAT]
    lo, hi, periodic = [0.0, 0.0, 0.0], list(L), (1, 1, 0 if slab else 1)
    if case["shape"] == "void":
        r2 = sum((pos[d] - 0.5 * L[d]) ** 2 for d in range(3))
        pos = pos[:, r2 >= case["void"] ** 2]
    elif case["shape"] == "vacancies":
        drop = torch.randperm(pos.shape[1], generator=g, device=device)[: max(1, pos.shape[1] // 216)]
        keep = torch.ones(pos.shape[1], dtype=torch.bool, device=device)
        keep[drop] = False
        pos = pos[:, keep]
    pos, noise = pos[:3].contiguous(), pos[3:]
    n = pos.shape[1]
    frozen = None
    if slab:
        lo[2], hi[2] = -10.0, float(pos[2].max().item()) + 10.0
        frozen = (pos[2] < 1.25 * A_LAT).to(torch.uint8)  # the bottom three (002) planes
    if frozen is not None:
        noise = noise * (frozen == 0)
    pos = pos + noise
    for d in range(3):
        if periodic[d]:
            pos[d] = torch.remainder(pos[d], L[d])
            pos[d][pos[d] >= hi[d]] = lo[d]
    vel = torch.randn((3, n), generator=g, device=device, dtype=torch.float64) * math.sqrt(KB * 300.0 / MASS * CONV)
    if frozen is not None:
        vel = vel * (frozen == 0)
    vel = vel - vel.mean(dim=1, keepdim=True) if frozen is None else vel
    return SimpleNamespace(pos=pos.contiguous(), lo=tuple(lo), hi=tuple(hi), periodic=periodic, frozen=frozen,
                           vel=vel.contiguous(), n=n, L=L)


def device_atoms(s):
    return ops.DeviceAtoms(s.pos, s.lo, s.hi, s.periodic, s.frozen)


# ------------------------------------------------------------------------------ cases
def block(cells, shape="vacancies", sigma=SIGMA_300, **more):
    nx, ny, nz = cells
    return dict(nx=nx, ny=ny, nz=nz, shape=shape, sigma=sigma, **more)


def listed():
    return [
        # the plain 6^3 block with vacancies: the smallest call, where launches count
        dict(name="eval_plain_860", kind="eval", n_max=8, l_max=3, anchored=False,
             **block((6, 6, 6), sigma=0.05)),
        # the void run's block under the closed-form fast potential
        dict(name="eam_void_130k", kind="eam", potential="closed", **block((32, 32, 32), "void", void=12.0)),
        # a larger block of uneven edges under the paper's copper potential
        dict(name="eam2_block_440k", kind="eam", potential="eam2", **block((47, 48, 49))),
        # the weights of the void run (Hyb1: thresholds 2.5/3.0, spreading 4/12 A)
        dict(name="weights_void_130k", kind="weights", **block((32, 32, 32), "void", void=12.0)),
        # double-precision ACE where the void run detects atoms
        dict(name="ace64_void", kind="ace", n_max=10, l_max=4, anchored=True,
             **block((32, 32, 32), "void", void=12.0)),
        # energy and forces of a 16^3 snapshot, as the differentiation runs take them
        dict(name="grad32_16k", kind="grad", precision="fp32", n_max=10, l_max=4, anchored=True,
             **block((16, 16, 16))),
        # a fitting step on one training structure
        dict(name="fit64_4k", kind="fit", precision="fp64", n_max=10, l_max=4, anchored=False,
             **block((10, 10, 10))),
        # the indicator's training: one mini-batch of the default size
        dict(name="train_4096", kind="train", batch=4096, pool=65536),
        # the indicator deployed on the void run's block
        dict(name="indicator_130k", kind="indicator", **block((32, 32, 32), "void", void=12.0)),
        # the void run: adaptive steps, weights every ten
        dict(name="md_void_130k", kind="md", steps=10, avg=0, thermostat=False, n_max=10, l_max=4, anchored=True,
             **block((32, 32, 32), "void", void=12.0)),
        # time-averaged weights and the local thermostat on a slab (the third sample, at step 20,
        # is the first that changes weights; the step after it corrects)
        dict(name="md_thermostat_256k", kind="md", steps=30, avg=11, thermostat=True, n_max=10, l_max=4,
             anchored=True, **block((40, 40, 40), "slab")),
        # the indentation block: the largest run
        dict(name="md_block_4m", kind="md", steps=10, avg=0, thermostat=False, n_max=10, l_max=4, anchored=True,
             **block((100, 100, 100), "slab")),
    ]


def draw(rng):
    def edges(lo, hi):
        """Three edges around one size drawn over its logarithm."""
        c = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        return tuple(max(lo, min(hi, int(round(c * rng.uniform(0.85, 1.18))))) for _ in range(3))

    def shape(least_void):
        s = rng.choice(["vacancies", "void", "slab"])
        return (s, dict(void=rng.uniform(4.0, least_void))) if s == "void" else (s, {})

    kind = rng.choice(["eval", "eam", "weights", "ace", "grad", "fit", "train", "indicator", "md"])
    sigma = rng.uniform(0.05, 0.1)
    if kind == "eval":
        s, more = shape(6.0)
        n_max, l_max = rng.choice([(8, 3), (6, 3), (10, 4), (9, 3)])
        return dict(kind=kind, n_max=n_max, l_max=l_max, anchored=rng.random() < 0.5,
                    **block(edges(4, 10), s, sigma, **more))
    if kind == "eam":
        s, more = shape(8.0)
        return dict(kind=kind, potential=rng.choice(["closed", "eam2"]), **block(edges(5, 48), s, sigma, **more))
    if kind == "weights":
        s, more = shape(12.0)
        return dict(kind=kind, **block(edges(8, 40), s, sigma, **more))
    if kind == "ace":
        s, more = shape(12.0)
        n_max, l_max = rng.choice([(8, 3), (10, 4), (7, 4), (12, 4), (12, 3)])
        return dict(kind=kind, n_max=n_max, l_max=l_max, anchored=rng.random() < 0.5,
                    **block(edges(8, 32), s, sigma, **more))
    if kind == "grad":
        s, more = shape(6.0)
        n_max, l_max = rng.choice([(8, 3), (10, 4), (9, 4), (12, 4)])
        return dict(kind=kind, precision=rng.choice(["fp32", "fp64"]), n_max=n_max, l_max=l_max,
                    anchored=rng.random() < 0.5, **block(edges(5, 18), s, sigma, **more))
    if kind == "fit":
        s, more = shape(6.0)
        n_max, l_max = rng.choice([(8, 3), (10, 4), (6, 4)])
        return dict(kind=kind, precision=rng.choice(["fp32", "fp64"]), n_max=n_max, l_max=l_max,
                    anchored=rng.random() < 0.5, **block(edges(4, 11), s, sigma, **more))
    if kind == "train":
        batch = int(round(math.exp(rng.uniform(math.log(200), math.log(16384)))))
        return dict(kind=kind, batch=batch, pool=4 * batch + 31)
    if kind == "indicator":
        s, more = shape(10.0)
        return dict(kind=kind, **block(edges(6, 44), s, sigma, **more))
    s, more = shape(12.0)
    avg = rng.choice([0, 0, 5, 11])
    return dict(kind=kind, steps=30 if avg else 10, avg=avg, thermostat=rng.random() < 0.3, n_max=10, l_max=4,
                anchored=True, **block(edges(12, 48), s, SIGMA_300, **more))


# ---------------------------------------------------------------------------- prepare
def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        return prepare_train(case, seed)
    s = crystal(case, seed)
    st = SimpleNamespace(case=case, s=s, ctx=ops.Context(0))
    st.atoms = device_atoms(s)
    if kind == "eval":
        st.model = ops.AceModel(st.ctx, ace_params(case["n_max"], case["l_max"], case["anchored"], seed))
    elif kind in ("weights", "indicator"):
        st.nl = ops.build_neighbors(st.ctx, st.atoms, 5.5)
        if kind == "indicator":
            st.csp = ops.compute_precision(st.ctx, st.atoms, st.nl, HYB1)["csp"]
            e = ops.eam_forces(st.ctx, st.atoms, st.nl, FAST)
            st.rho, st.f = e["rho"], e["f"]
            st.net = ops.Mlp(st.ctx, learned.glorot_params(int(seed)), [9.0, 1.5, 12.0, 0.7], [0.8, 1.5, 0.6, 0.5])
            st.net.set_range([5.0, 0.0, 7.0, 0.0], [14.0, 40.0, 15.0, 6.0])
    elif kind == "ace":
        st.model = ops.AceModel(st.ctx, ace_params(case["n_max"], case["l_max"], case["anchored"], seed))
        st.nl = ops.build_neighbors(st.ctx, st.atoms, 5.5)
        pr = ops.compute_precision(st.ctx, st.atoms, st.nl, HYB1)
        st.w, st.active = pr["w"], pr["active"].clone()
    elif kind in ("grad", "fit"):
        prm = ace_params(case["n_max"], case["l_max"], case["anchored"], seed)
        st.model = ops.AceModel(st.ctx, prm)
        st.runner = autograd.AceRunner(st.ctx, st.model, s.lo, s.hi, s.periodic, precision=case["precision"])
        dt = torch.float32 if case["precision"] == "fp32" else torch.float64
        st.dtype = dt
        if kind == "grad":
            st.pos = s.pos.to(dt).requires_grad_(True)
            st.c1, st.c2 = torch.from_numpy(prm.c1), torch.from_numpy(prm.c2)
        else:
            st.c1 = torch.from_numpy(prm.c1).to("cuda", dt).requires_grad_(True)
            st.c2 = torch.from_numpy(prm.c2).to("cuda", dt).requires_grad_(True)
    elif kind == "md":
        st.model = ops.AceModel(st.ctx, ace_params(case["n_max"], case["l_max"], case["anchored"], seed))
        ind = None
        if case["shape"] == "slab":
            top = s.hi[2] - 10.0
            ind = dict(radius=40.0, k=10.0, center=[0.5 * s.L[0], 0.5 * s.L[1], top + 40.0], velocity=[0.0, 0.0, -0.2])
        th = dict(r_omega=13.5, omega_max=800, seed=2024) if case["thermostat"] else None
        st.md = ops.MD(st.ctx, st.atoms, FAST, st.model, HYB1, dt=1e-3, skin=0.5, max_nb=80, precision_every=10,
                       ace_precision="fp32", mode="adaptive", indenter=ind, avg_samples=case["avg"],
                       avg_dw_min=1.0 / max(1, case["avg"]), thermostat=th)
    return st


def train_data(case, seed):
    """Features and labels with the distributions the training structures give."""
    rng = np.random.default_rng(int(seed))
    n = case["pool"]
    csp = rng.gamma(2.0, 0.45, n)
    feat = np.stack([rng.normal(9.0, 0.8, n), csp, np.rint(rng.normal(12.0, 0.6, n)), rng.gamma(2.0, 0.35, n)], axis=1)
    label = -4.0 + 0.8 * np.log1p(csp) + 0.5 * feat[:, 3] - 0.1 * (feat[:, 0] - 9.0) + rng.normal(0.0, 0.25, n)
    sel = rng.choice(n, size=case["batch"], replace=False)
    feat = feat.astype(np.float32)
    params = learned.glorot_params(int(seed))
    mu, sd = feat.mean(axis=0, dtype=np.float64), feat.std(axis=0, dtype=np.float64)
    return feat, label.astype(np.float32), sel.astype(np.int32), params, mu.astype(np.float32), sd.astype(np.float32)


def prepare_train(case, seed):
    feat, label, sel, params, mu, sd = train_data(case, seed)
    st = SimpleNamespace(case=case, ctx=ops.Context(0))
    st.feat, st.label, st.sel = (torch.from_numpy(v).cuda() for v in (feat, label, sel))
    st.net = ops.Mlp(st.ctx, params, mu, sd)
    return st


# -------------------------------------------------------------------------------- run
def run(st):
    kind = st.case["kind"]
    if kind == "eval":
        nl = ops.build_neighbors(st.ctx, st.atoms, 5.5)
        pr = ops.compute_precision(st.ctx, st.atoms, nl, PLAIN)
        e = ops.eam_forces(st.ctx, st.atoms, nl, FAST, pr["w"])
        a = ops.ace_energy_forces(st.ctx, st.atoms, nl, st.model, pr["active"], pr["w"], precision="fp64")
        b = ops.blend(st.ctx, pr["w"], e["e_site"], a["e_site"], e["f"], a["f"])
        return dict(w=pr["w"], mask=pr["mask"], e_site=b["e_site"], f=b["f"], e_pot=b["e_pot"])
    if kind == "eam":
        closed_form = st.case["potential"] == "closed"
        nl = ops.build_neighbors(st.ctx, st.atoms, 5.5 if closed_form else 6.0, max_nb=80 if closed_form else 96)
        e = ops.eam_forces(st.ctx, st.atoms, nl, FAST if closed_form else EAM2)
        return dict(count=nl.count, e_site=e["e_site"], rho=e["rho"], f=e["f"])
    if kind == "weights":
        pr = ops.compute_precision(st.ctx, st.atoms, st.nl, HYB1)
        return dict(csp=pr["csp"], w0=pr["w0"], w=pr["w"], mask=pr["mask"], n_active=pr["n_active"])
    if kind == "ace":
        a = ops.ace_energy_forces(st.ctx, st.atoms, st.nl, st.model, st.active, st.w, precision="fp64")
        return dict(e_site=a["e_site"], f=a["f"])
    if kind == "grad":
        st.pos.grad = None
        e = autograd.ace_energy(st.pos.double(), st.c1, st.c2, st.runner).to(st.dtype)
        e.backward()
        return dict(e=e.detach(), grad=st.pos.grad)
    if kind == "fit":
        st.c1.grad = st.c2.grad = None
        n = st.s.n
        e = autograd.ace_energy(st.s.pos, st.c1.double(), st.c2.double(), st.runner).to(st.dtype)
        (((e + 3.4 * n) / n) ** 2).backward()
        with torch.no_grad():
            st.c1.add_(st.c1.grad, alpha=-1e-6)
            st.c2.add_(st.c2.grad, alpha=-1e-6)
        return dict(e=e.detach(), g1=st.c1.grad, g2=st.c2.grad)
    if kind == "train":
        g, loss = st.net.gradients(st.feat, st.label, st.sel)
        return dict(grad=g, loss=loss)
    if kind == "indicator":
        feat = ops.features(st.ctx, st.atoms, st.nl, st.rho, st.csp, st.f)
        pred, w0 = st.net.precision(feat, 0.004, 0.008)
        return dict(feat=feat, pred=pred, w0=w0)
    # a segment of a trajectory from a restart point: forces and weights there, then the steps
    pos, vel = st.s.pos.clone(), st.s.vel.clone()
    f, w = st.md.init(pos)
    out = st.md.step(pos, vel, f, w, st.case["steps"], allow_radicand=True)
    # the frame a trajectory file and its log take: the positions as they are, and velocities,
    # forces, weights and energies in single precision (they come from float32 ACE)
    return dict(pos=pos, vel=vel.float(), f=f.float(), w=w.float(), e_pot=np.float32(out["e_pot"]),
                e_kin=np.float32(out["e_kin"]))


# ------------------------------------------------------------------------------- work
@functools.lru_cache(maxsize=None)
def ace_flops(n_max, l_max, coefficients):
    """Per evaluated atom with 42 neighbours inside the cutoff: atomic base, products and
    their adjoint (about 70 operations a triple when the pairs are coupled first), force."""
    lm = (l_max + 1) ** 2
    nb = 42.0
    base = nb * (3 * n_max + 4 * lm + 2 * n_max * lm) + 2.0 * n_max * n_max * lm
    force = nb * (4 * n_max * lm + 12 * lm + 6 * n_max) + 2.0 * n_max * n_max * lm
    return base + force + (80.0 if coefficients else 70.0) * len(triples(n_max, l_max))


def atoms_of(case):
    n = 4.0 * case["nx"] * case["ny"] * case["nz"]
    return n - 4.19 * case["void"] ** 3 * 4 / A_LAT ** 3 if case["shape"] == "void" else n


def active_of(case, n):
    """Roughly how many atoms the criterion detects: the void's or the surface's shell of
    12 A, and the thermal outliers' neighbourhoods."""
    if case["shape"] == "void":
        shell = 4.19 * ((case["void"] + 14.0) ** 3 - case["void"] ** 3) * 4 / A_LAT ** 3
    elif case["shape"] == "slab":
        shell = 4.0 * case["nx"] * case["ny"] * 12.0 / A_LAT
    else:
        shell = n / 216.0 * 300.0
    return min(n, shell + 0.02 * n)


def work(case):
    kind = case["kind"]
    if kind == "train":
        return dict(bytes=case["batch"] * 24.0 + 4.0 * 8705 * 2, flops=case["batch"] * 6.0 * 8512)
    n = atoms_of(case)
    nb = 55.0
    if kind == "eam":
        return dict(bytes=n * (24.0 + 4.0 + 40.0), flops=n * nb * 90.0)
    if kind == "weights":
        return dict(bytes=n * (4.0 * (1 + nb) + 24.0 + 24.0 + 5.0), flops=n * (nb * 10.0 + 66 * 12.0))
    if kind == "indicator":
        return dict(bytes=n * (4.0 * (1 + nb) + 24.0 + 40.0 + 28.0), flops=n * 17000.0)
    if kind in ("grad", "fit"):
        return dict(bytes=n * (24.0 + 24.0), flops=n * ace_flops(case["n_max"], case["l_max"], kind == "fit"))
    if kind == "eval":
        return dict(bytes=n * (24.0 + 40.0), flops=n * (ace_flops(case["n_max"], case["l_max"], False) + nb * 110.0))
    act = active_of(case, n)
    if kind == "ace":
        return dict(bytes=n * 40.0 + act * (24.0 + 4.0 * nb), flops=act * ace_flops(case["n_max"], case["l_max"], False))
    k = case["steps"] + 1
    return dict(bytes=k * n * (4.0 * nb + 24.0 * 4 + 40.0),
                flops=k * (n * nb * 90.0 + act * ace_flops(case["n_max"], case["l_max"], False)))


# ------------------------------------------------------- the same in plain 64-bit torch
def windows(s, reach, chunk):
    """Yields (rows, candidates): atoms in order of x, a chunk at a time, with the atoms
    whose x lies within ``reach`` of the chunk's (minimum image)."""
    x = s.pos[0]
    order = torch.argsort(x)
    L = s.hi[0] - s.lo[0]
    for k in range(0, s.n, chunk):
        rows = order[k:k + chunk]
        a, b = x[rows].min(), x[rows].max()
        mid, half = 0.5 * (a + b), 0.5 * (b - a) + reach
        d = x - mid
        if s.periodic[0]:
            d = d - L * torch.round(d / L)
        yield rows, torch.nonzero(d.abs() <= half).reshape(-1)


def separation(s, rows, cand):
    out = []
    for d in range(3):
        v = s.pos[d][cand][None, :] - s.pos[d][rows][:, None]
        if s.periodic[d]:
            L = s.hi[d] - s.lo[d]
            v = v - L * torch.round(v / L)
        out.append(v)
    return out


def pair_list(s, rc):
    """All ordered pairs (i, j) closer than rc, and the lattice shift of each."""
    ii, jj = [], []
    for rows, cand in windows(s, rc, 1024):
        dx, dy, dz = separation(s, rows, cand)
        hit = (dx * dx + dy * dy + dz * dz < rc * rc) & (rows[:, None] != cand[None, :])
        a, b = torch.nonzero(hit, as_tuple=True)
        ii.append(rows[a])
        jj.append(cand[b])
    i, j = torch.cat(ii), torch.cat(jj)
    shift = torch.zeros((3, i.numel()), dtype=torch.float64, device=s.pos.device)
    for d in range(3):
        if s.periodic[d]:
            L = s.hi[d] - s.lo[d]
            shift[d] = -L * torch.round((s.pos[d][j] - s.pos[d][i]) / L)
    return i, j, shift


def psi(x):
    x4 = x ** 4
    return torch.where(x < 0, x4 / (1 + x4), torch.zeros_like(x))


def eam_sites(r, i, n, p):
    """(site energy, density) of the pairs at distances r."""
    t = psi((r - p.rc) / p.h)
    if hasattr(p, "xi0"):
        m = lambda r0, al: torch.exp(-2 * al * (r - r0)) - 2 * torch.exp(-al * (r - r0))  # noqa: E731
        phi = (p.E1 * m(p.r01, p.alpha1) + p.E2 * m(p.r02, p.alpha2) + p.delta) * t
        for S, rs in zip(p.S, p.rs):
            phi = phi - S * torch.clamp(rs - r, min=0.0) ** 4
        rho_p = (p.a * torch.exp(-p.beta1 * (r - p.r03) ** 2) + torch.exp(-p.beta2 * (r - p.r04))) * t
    else:
        phi = p.A * torch.exp(-p.alpha * (r - p.r0)) * t
        rho_p = torch.exp(-p.beta * (r - p.r0)) * t
    zero = torch.zeros(n, dtype=r.dtype, device=r.device)
    rho, pair = zero.index_add(0, i, rho_p), zero.index_add(0, i, phi)
    if hasattr(p, "xi0"):
        x = rho - 1.0
        low = p.xi0 + 0.5 * p.xi2 * x ** 2 + sum(q * x ** (k + 3) for k, q in enumerate(p.q))
        high = (p.xi0 + 0.5 * p.xi2 * x ** 2 + p.q[0] * x ** 3 + p.Q1 * x ** 4) / (1 + p.Q2 * x ** 3)
        F = torch.where(rho <= 1.0, low, high) + p.f0
    else:
        F = -torch.sqrt(rho)
    return F + 0.5 * pair, rho


def exact_csp(s, prec):
    csp = torch.full((s.n,), math.inf, dtype=torch.float64, device=s.pos.device)
    up = torch.triu_indices(12, 12, 1, device=s.pos.device)
    for rows, cand in windows(s, prec.r_cut, 512):
        d = separation(s, rows, cand)
        r2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2
        r2[rows[:, None] == cand[None, :]] = math.inf
        r2[r2 >= prec.r_cut ** 2] = math.inf
        best, at = torch.topk(r2, 12, dim=1, largest=False)
        v = torch.stack([torch.gather(x, 1, at) for x in d], dim=2)
        sq = ((v[:, up[0]] + v[:, up[1]]) ** 2).sum(dim=2)
        c = torch.topk(sq, 6, dim=1, largest=False).values.sum(dim=1)
        csp[rows] = torch.where(torch.isinf(best[:, 11]), torch.full_like(c, math.inf), c)
    if s.frozen is not None:
        csp[s.frozen != 0] = 0.0
    return csp


def f_cut(x):
    y = 1.0 - 1.875 * x + 1.25 * x ** 3 - 0.375 * x ** 5
    return torch.where(x < 0, torch.ones_like(x), torch.where(x > 1, torch.zeros_like(x), y))


def exact_weights(s, prec):
    csp = exact_csp(s, prec)
    x = (csp - prec.csp_lo) / (prec.csp_hi - prec.csp_lo)
    x = torch.clamp(x, -1.0, 2.0)
    w0 = torch.clamp(x, 0.0, 1.0) if prec.switch_kind == 0 else 1.0 - f_cut(x)
    if s.frozen is not None:
        w0[s.frozen != 0] = 0.0
    w = w0.clone()
    if prec.r_hi > 0:
        for rows, cand in windows(s, prec.r_hi, 1024):
            src = cand[w0[cand] > 0]
            if not src.numel():
                continue
            for k in range(0, src.numel(), 4096):
                c = src[k:k + 4096]
                d = separation(s, rows, c)
                r = torch.sqrt(d[0] ** 2 + d[1] ** 2 + d[2] ** 2)
                v = w0[c][None, :] * f_cut((r - prec.r_lo) / (prec.r_hi - prec.r_lo))
                v = torch.where(r < prec.r_hi, v, torch.zeros_like(v))
                w[rows] = torch.maximum(w[rows], v.max(dim=1).values)
        if s.frozen is not None:
            w[s.frozen != 0] = 0.0
    return csp, w0, w


def harmonics(u, l_max):
    """Real orthonormal spherical harmonics of unit vectors u [P, 3]: [P, (l_max + 1)^2]."""
    x, y, z = u[:, 0], u[:, 1], u[:, 2]
    re, im = [torch.ones_like(x)], [torch.zeros_like(x)]
    for _ in range(l_max):
        re, im = re + [re[-1] * x - im[-1] * y], im + [re[-1] * y + im[-1] * x]
    cols = []
    for l in range(l_max + 1):
        for m in range(-l, l + 1):
            k = abs(m)
            poly = np.polynomial.polynomial.polyder(np.polynomial.legendre.leg2poly([0.0] * l + [1.0]), k)
            q = torch.zeros_like(z)
            for c in reversed(np.atleast_1d(poly)):
                q = q * z + float(c)
            norm = math.sqrt((2 * l + 1) / (4 * math.pi) * math.factorial(l - k) / math.factorial(l + k))
            cols.append(norm * q * (1.0 if m == 0 else math.sqrt(2.0) * (re[k] if m > 0 else im[k])))
    return torch.stack(cols, dim=1)


@functools.lru_cache(maxsize=None)
def gaunt(l_max):
    """Integrals of three real harmonics over the sphere, by an exact product rule."""
    xs, ws = np.polynomial.legendre.leggauss(2 * l_max + 2)
    k = 3 * l_max + 3
    ph = np.arange(k) * (2 * np.pi / k)
    z, f = np.repeat(xs, k), np.tile(ph, xs.size)
    q = np.sqrt(1 - z * z)
    Y = harmonics(torch.from_numpy(np.stack([q * np.cos(f), q * np.sin(f), z], axis=1)), l_max).numpy()
    wt = np.repeat(ws, k) * (2 * np.pi / k)
    return np.einsum("q,qa,qb,qc->abc", wt, Y, Y, Y, optimize=True)


def third_order(A, c, n_max, l_max):
    """sum over the third-order functions of c . B for A [i, n_max, (l_max + 1)^2]."""
    G = torch.from_numpy(gaunt(l_max)).to(A.device)
    sl = [slice(l * l, (l + 1) * (l + 1)) for l in range(l_max + 1)]
    total = 0.0
    for (l1, l2, l3), C in c.items():
        X, Y, Z = A[:, :, sl[l1]], A[:, :, sl[l2]], A[:, :, sl[l3]]
        i, n = X.shape[0], n_max
        n1, n2, n3 = 2 * l1 + 1, 2 * l2 + 1, 2 * l3 + 1
        XY = (X[:, :, None, :, None] * Y[:, None, :, None, :]).reshape(i * n * n, n1 * n2)
        P = (XY @ G[sl[l1], sl[l2], sl[l3]].reshape(n1 * n2, n3)).reshape(i, n * n, n3)
        D = (Z.permute(0, 2, 1).reshape(i * n3, n) @ C.reshape(n * n, n).T.contiguous()).reshape(i, n3, n * n)
        total = total + (P * D.permute(0, 2, 1)).sum(dim=(1, 2))
    return total


def dense(c, n_max, l_max, device):
    """The coefficient vector c of the basis as tensors: first, second and third order."""
    LL = l_max + 1
    b1 = c[:n_max]
    k = n_max
    at2 = torch.zeros((n_max, n_max, LL), dtype=torch.int64)
    for n1 in range(n_max):
        for n2 in range(n1, n_max):
            for l in range(LL):
                at2[n1, n2, l] = k + 1
                k += 1
    at3 = {}
    for (n1, l1), (n2, l2), (n3, l3) in triples(n_max, l_max):
        t = at3.setdefault((l1, l2, l3), np.zeros((n_max,) * 3, dtype=np.int64))
        t[n1, n2, n3] = k + 1
        k += 1
    padded = torch.cat([torch.zeros(1, dtype=c.dtype, device=c.device), c])
    return b1, padded[at2.to(device)], {key: padded[torch.from_numpy(v).to(device)] for key, v in at3.items()}


def atomic_base(s, pos, i, j, shift, prm, row, m):
    d = pos[:, j] - pos[:, i] + shift
    r = torch.sqrt((d * d).sum(dim=0))
    x = 2.0 * r / prm.rc - 1.0
    T = [torch.ones_like(x), x]
    for _ in range(2, prm.n_max):
        T.append(2.0 * x * T[-1] - T[-2])
    g = torch.stack(T[:prm.n_max], dim=1) * psi((r - prm.rc) / prm.h)[:, None]
    Y = harmonics((d / r).T, prm.l_max)
    W = torch.from_numpy(prm.W).to(pos.device)
    A = torch.zeros((m, prm.n_max, (prm.l_max + 1) ** 2), dtype=torch.float64, device=pos.device)
    parts = []
    for l in range(prm.l_max + 1):
        a, b = l * l, (l + 1) * (l + 1)
        v = (g @ W[l].T)[:, :, None] * Y[:, None, a:b] / prm.s_a
        parts.append(v)
    return A.index_add(0, row[i], torch.cat(parts, dim=2)), r


def exact_ace(s, prm, active, w, want_c=False):
    """(site energies of ``active``, forces of sum w_i E_i, dE/dc1, dE/dc2)."""
    dev = s.pos.device
    i, j, shift = pair_list(s, prm.rc)
    row = torch.full((s.n,), -1, dtype=torch.int64, device=dev)
    row[active] = torch.arange(active.numel(), device=dev)
    keep = row[i] >= 0
    i, j, shift = i[keep], j[keep], shift[:, keep]
    order = torch.argsort(row[i])
    i, j, shift = i[order], j[order], shift[:, order]
    c = [torch.from_numpy(v).to(dev).requires_grad_(want_c) for v in (prm.c1, prm.c2)]
    grad_pos = torch.zeros_like(s.pos)
    grad_c = [torch.zeros_like(v) for v in c]
    e_act = torch.zeros(active.numel(), dtype=torch.float64, device=dev)
    first = torch.searchsorted(row[i].contiguous(), torch.arange(active.numel() + 1, device=dev))
    for k in range(0, active.numel(), 2048):
        m = min(2048, active.numel() - k)
        a, b = int(first[k]), int(first[k + m])
        ii, jj, sh = i[a:b], j[a:b], shift[:, a:b]
        local = row - k
        pos = s.pos.clone().requires_grad_(True)
        A, r = atomic_base(s, pos, ii, jj, sh, prm, local, m)
        phi = []
        for cv in c:
            b1, b2, b3 = dense(cv, prm.n_max, prm.l_max, dev)
            v = A[:, :, 0] @ b1
            for l in range(prm.l_max + 1):
                X = A[:, :, l * l:(l + 1) ** 2]
                v = v + ((X.permute(0, 2, 1).reshape(-1, prm.n_max) @ b2[:, :, l]).reshape(m, 2 * l + 1, prm.n_max)
                         * X.permute(0, 2, 1)).sum(dim=(1, 2))
            phi.append(v + third_order(A, b3, prm.n_max, prm.l_max))
        ax = phi[1].abs()
        e = phi[0] + torch.sign(phi[1]) * (torch.sqrt(ax + prm.eps ** 2) - prm.eps)
        if prm.anchor is not None:
            e = e + eam_sites(r, local[ii], m, prm.anchor)[0]
        e_act[k:k + m] = e.detach()
        weight = w[active[k:k + m]] if w is not None else torch.ones_like(e)
        got = torch.autograd.grad((weight * e).sum(), [pos] + (c if want_c else []))
        grad_pos += got[0]
        for x, y in zip(grad_c, got[1:]):
            x += y
    return e_act, -grad_pos, grad_c[0], grad_c[1]


def exact_eam(s, p, w, rc):
    i, j, shift = pair_list(s, rc)
    pos = s.pos.clone().requires_grad_(True)
    d = pos[:, j] - pos[:, i] + shift
    e, rho = eam_sites(torch.sqrt((d * d).sum(dim=0)), i, s.n, p)
    u = torch.ones_like(e) if w is None else 1.0 - w
    (g,) = torch.autograd.grad((u * e).sum(), pos)
    return e.detach(), rho.detach(), -g


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return exact_train(case, seed)
    if kind == "md":
        return None
    s = crystal(case, seed)
    if kind == "eam":
        p = FAST if case["potential"] == "closed" else EAM2
        e, rho, f = exact_eam(s, p, None, p.rc)
        return dict(count=None, e_site=e, rho=rho, f=f)
    if kind == "weights":
        csp, w0, w = exact_weights(s, HYB1)
        return dict(csp=csp, w0=w0, w=w, mask=None, n_active=None)
    if kind == "indicator":
        csp = torch.clamp(exact_csp(s, HYB1), max=50.0)
        _, rho, f = exact_eam(s, FAST, None, RC)
        i, _, _ = pair_list(s, 3.08)
        feat = torch.stack([rho, csp, torch.bincount(i, minlength=s.n).double(), f.norm(dim=0)], dim=1)
        return dict(feat=feat, pred=None, w0=None)
    prm = ace_params(case["n_max"], case["l_max"], case["anchored"], seed)
    every = torch.arange(s.n, device=s.pos.device)
    if kind == "grad":
        if case["precision"] == "fp32":
            s.pos = s.pos.float().double()
        e, f, _, _ = exact_ace(s, prm, every, None)
        return dict(e=e.sum(), grad=-f)
    if kind == "fit":
        if case["precision"] == "fp32":
            prm.c1, prm.c2 = (v.astype(np.float32).astype(np.float64) for v in (prm.c1, prm.c2))
        e, _, g1, g2 = exact_ace(s, prm, every, None, want_c=True)
        total = e.sum()
        slope = 2.0 * (total + 3.4 * s.n) / s.n ** 2
        return dict(e=total, g1=slope * g1, g2=slope * g2)
    prec = PLAIN if kind == "eval" else HYB1
    _, _, w = exact_weights(s, prec)
    active = torch.nonzero(w > 0).reshape(-1)
    e_act, f, _, _ = exact_ace(s, prm, active, w)
    e_ace = torch.zeros(s.n, dtype=torch.float64, device=s.pos.device)
    e_ace[active] = e_act
    if kind == "ace":
        return dict(e_site=e_ace, f=f)
    e, _, f_eam = exact_eam(s, FAST, w, RC)
    site = (1.0 - w) * e + w * e_ace
    return dict(w=w, mask=None, e_site=site, f=f + f_eam, e_pot=site.sum().reshape(1))


def exact_train(case, seed):
    feat, label, sel, params, mu, sd = train_data(case, seed)
    at = np.cumsum([0, 256, 64, 4096, 64, 4096, 64, 64, 1])
    p = torch.from_numpy(params.astype(np.float64)).requires_grad_(True)
    W1, b1, W2, b2, W3, b3, W4, b4 = (p[at[k]:at[k + 1]] for k in range(8))
    x = (torch.from_numpy(feat[sel]).double() - torch.from_numpy(mu).double()) / torch.from_numpy(sd).double()
    h = torch.tanh(x @ W1.reshape(64, 4).T + b1)
    h = torch.tanh(h @ W2.reshape(64, 64).T + b2)
    h = torch.tanh(h @ W3.reshape(64, 64).T + b3)
    loss = ((h @ W4 + b4 - torch.from_numpy(label[sel]).double()) ** 2).mean()
    (g,) = torch.autograd.grad(loss, p)
    return dict(grad=g, loss=loss.detach().reshape(1))

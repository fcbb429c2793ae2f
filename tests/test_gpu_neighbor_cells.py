"""Neighbour rows where the build changes its way: cells per axis (images found per pair below five),
blocks shared by a cell's atoms or not, rows of one and of two keys per lane, pairs at the list radius to
rounding, positions outside the periodic box, more entries than a row keeps.  Rows are whole numbers:
equal to the oracle's, entry for entry.
"""

import numpy as np
import pytest
import torch

import synth
from oracle import geometry
from synth import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import ops
    return ops, ops.Context(0)


def gas(box, density, periodic, seed):
    box = np.asarray(box, dtype=float)
    rng = np.random.default_rng(seed)
    n = int(density * box.prod())
    lo = np.array([-3.0, 1.5, 0.0])
    return synth.System(lo[:, None] + rng.uniform(0.0, 1.0, (3, n)) * box[:, None], lo, lo + box, periodic)


def check(ops, ctx, s, r_list, max_nb=128):
    nl = ops.build_neighbors(ctx, ops.device_atoms(s), r_list, max_nb=max_nb)
    off, idx = geometry.neighbor_csr(s.pos, s.lo, s.hi, s.periodic, r_list)
    cnt, rows = nl.count.cpu().numpy(), nl.idx.cpu().numpy()
    assert np.array_equal(cnt, np.diff(off))
    assert np.array_equal(rows[:max_nb].T[np.arange(max_nb)[None, :] < cnt[:, None]], idx)
    assert nl.needed == np.diff(off).max()
    return cnt


@pytest.mark.parametrize("box,density,periodic,r_list", [
    ((8.0, 9.0, 40.0), 0.05, (0, 0, 0), 5.5),      # one cell on two axes, open
    ((11.2, 17.0, 22.1), 0.09, (1, 1, 1), 5.5),    # two, three and four cells
    ((28.0, 33.1, 11.2), 0.06, (1, 1, 0), 5.5),    # five, six and two
    ((61.0, 56.0, 27.6), 0.085, (1, 0, 1), 5.5),
    ((66.5, 72.0, 78.5), 0.06, (1, 1, 1), 6.5),   # rows past 64 entries, 1,210 cells
])
def test_gas(env, box, density, periodic, r_list):
    ops, ctx = env
    print(f"[case] gas {box} {periodic}", flush=True)
    check(ops, ctx, gas(box, density, periodic, 7), r_list)


@pytest.mark.parametrize("cells", [4, 9])
def test_pairs_at_the_list_radius(env, cells):
    """A static crystal and a list radius equal to a shell's distance: every row has pairs that float32
    cannot place."""
    ops, ctx = env
    print(f"[case] shell radius, {cells} cells", flush=True)
    s = configs.bulk(cells, seed=2, vacancies=3)
    a = (s.hi - s.lo)[0] / cells
    check(ops, ctx, s, float(a * np.sqrt(2.5)))


def test_outside_the_box(env):
    """Atoms that left a periodic box by up to 0.7 A and were not wrapped (cells 0.9 A wider than the
    list radius still hold every pair)."""
    ops, ctx = env
    print("[case] outside the box", flush=True)
    s = gas((38.4, 38.4, 38.4), 0.07, (1, 1, 1), 5)
    rng = np.random.default_rng(8)
    move = rng.uniform(-0.7, 0.7, s.pos.shape)
    check(ops, ctx, synth.System(s.pos + move, s.lo, s.hi, s.periodic), 5.5)


@pytest.mark.parametrize("density", [0.19, 0.45])
def test_rows_too_long(env, density):
    """Rows past the 128 entries a list can have, and past what a wave keeps while it looks."""
    ops, ctx = env
    print(f"[case] density {density}", flush=True)
    from paper_2411_03002_amd import binding
    s = gas((20.0, 28.0, 30.0), density, (1, 1, 1), 6)
    off, _ = geometry.neighbor_csr(s.pos, s.lo, s.hi, s.periodic, 5.5)
    with pytest.raises(binding.ApxError) as err:
        ops.build_neighbors(ctx, ops.device_atoms(s), 5.5, max_nb=128, grow=False)
    assert f"row of {np.diff(off).max()} entries" in str(err.value)

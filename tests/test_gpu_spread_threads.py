"""The spread weight where the number of threads per source changes (8,192 sources): bit-equal to the
oracle's, as elsewhere (maxima do not depend on the order of the sources).
"""

import numpy as np
import pytest
import torch

import synth
from oracle import precision
from synth import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 37, 8192, 8193])
def test_sources(k):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import ops
    print(f"[case] {k} sources", flush=True)
    s = configs.bulk(14, seed=14, temperature=300.0, vacancies=5)
    prm = synth.PrecisionParams(2.5, 3.0, 1, 4.0, 6.0)
    rng = np.random.default_rng(k)
    csp = np.zeros(s.n)
    csp[rng.choice(s.n, k, replace=False)] = rng.uniform(2.51, 3.5, k)
    ctx = ops.Context(0)
    atoms = ops.device_atoms(s)
    nl = ops.build_neighbors(ctx, atoms, 5.5)
    got = ops.compute_precision(ctx, atoms, nl, prm, csp=torch.as_tensor(csp, device="cuda"))
    w0, w = got["w0"].cpu().numpy(), got["w"].cpu().numpy()
    src = np.flatnonzero(w0 > 0.0)
    assert src.size == k
    want = precision.spread(s.pos, s.lo, s.hi, s.periodic, w0, prm.r_lo, prm.r_hi)
    assert np.array_equal(w, want)

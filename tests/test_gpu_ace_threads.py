"""Two host threads, a context each, with models of 11 and 12 radial functions, which share the kernels'
instantiations but not their LDS sizes: every call succeeds and gives the bits it gives alone."""

import threading

import pytest
import torch

import synth
from oracle import ace as oace
from synth import configs

pytestmark = pytest.mark.gpu


def test_models_of_one_instantiation_in_two_threads():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2411_03002_amd import ops
    print("[case] two threads, n_max 11 and 12", flush=True)
    s = configs.bulk(6, seed=2, sigma=0.08)

    def call(n_max):
        ctx = ops.Context(0)
        atoms = ops.device_atoms(s)
        nl = ops.build_neighbors(ctx, atoms, 5.5)
        model = ops.AceModel(ctx, synth.ace_random(n_max, 4, oace.num_basis(n_max, 4), seed=3))
        active = torch.arange(s.n, dtype=torch.int32, device="cuda")
        return lambda p: ops.ace_energy_forces(ctx, atoms, nl, model, active, None, p, want_dc=True)

    keys = ("e_site", "dE_dc1", "dE_dc2")
    calls = {n: call(n) for n in (11, 12)}
    ref = {n: {p: calls[n](p) for p in ("fp32", "fp64")} for n in calls}
    torch.cuda.synchronize()
    bad, done = [], {11: 0, 12: 0}

    def work(n):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for k in range(150):
                    p = "fp32" if k % 2 else "fp64"
                    out = calls[n](p)
                    torch.cuda.current_stream().synchronize()
                    if not all(torch.equal(out[x], ref[n][p][x]) for x in keys):
                        bad.append((n, k))
                    done[n] += 1
        except Exception as e:  # noqa: BLE001
            bad.append((n, repr(e)))

    threads = [threading.Thread(target=work, args=(n,)) for n in calls]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad[:3]
    assert done == {11: 150, 12: 150}

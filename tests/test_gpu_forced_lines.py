"""The forced step over the line solvers its sweeps can take: partitioned
lines with wall data on every side, r or theta lines past 256 rows two-ended
with the scalar lines apart (a multiple of 8 rows) or together, several slots
per phi workgroup and one, with every forcing input.  Bar: the forced tests'
1e-11 relative L2 per field against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import compare
from helpers import random_state, random_wall
from paper_2004_13887_amd import inputs as I

pytestmark = pytest.mark.gpu

SPECS = [I.sector(4, 264, 5, 4e-4, 5e-4), I.sector(3, 261, 4, 4e-4, 5e-4), I.sector(264, 4, 5, 4e-4, 5e-4),
         I.sector(7, 33, 12, 4e-4, 5e-4), I.sector(3, 5, 260, 4e-4, 5e-4), I.full_sphere(12, 17, 64)]


@pytest.mark.parametrize("spec", SPECS, ids=lambda g: f"{g.nr}x{g.nt}x{g.np}")
def test_forced_step_line_solvers(spec):
    from paper_2004_13887_amd import dsw
    print(f"[forced lines] {spec.nr}x{spec.nt}x{spec.np}", flush=True)
    U0, tau = random_state(spec, 901, mach=0.05)
    rng = np.random.Generator(np.random.PCG64(902))
    scale = {"p": 1e-4 * np.mean(U0["p"]), "ur": 1.0, "ut": 1.0, "uf": 1.0, "T": 1e-3 * np.mean(U0["T"])}
    src = {k: scale[k] * rng.uniform(-1.0, 1.0, v.shape) for k, v in U0.items()}
    bnd = {k: U0[k] + rng.uniform(-2.0, 2.0, U0[k].shape) for k in ("ur", "ut", "uf")}
    w0, w1 = random_wall(spec, 903, scale=3.0), random_wall(spec, 904, scale=3.0)
    full = dict(bnd, p=U0["p"], T=U0["T"])
    ref = oracle.split_step(oracle.Grid(*spec.args()), oracle.Material(*I.AIR.astuple()), U0, tau, 2, wall0=w0,
                            wall1=w1, src=src, bnd=full)
    gg = dsw.Grid.from_spec(spec, I.AIR)
    out = gg.empty()
    gg.split_step_forced(dsw.to_device(U0), out, tau, 2, src=dsw.to_device(src), wall0=dsw.to_device(w0),
                         wall1=dsw.to_device(w1), bnd=dsw.to_device(full))
    torch.cuda.synchronize()
    gg.get_status()
    e = compare("forced lines", dsw.to_host(out), ref, base=U0)
    assert max(e[k] for k in U0) <= 1e-11

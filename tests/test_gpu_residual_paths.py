"""The public residual on both sides of the size where it writes the midpoint
first: the last grid of the one-launch form, the first of the two-step form,
sector and sphere, on arrays that start at an odd multiple of 8 bytes.  Bar:
the parity tests' 1e-11 relative L2 (the u_r row against tau g, as there);
the midpoint is exact (one rounding on either side)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2004_13887_amd import inputs as I
from test_gpu_parity import residual_errors

pytestmark = pytest.mark.gpu

GRIDS = {"sector-one-launch": I.sector(40, 41, 65, 4e-4, 5e-4), "sector-two-step": I.sector(40, 42, 65, 4e-4, 5e-4),
         "sphere-two-step": I.full_sphere(40, 43, 67)}


@pytest.mark.parametrize("odd", [0, 1])
@pytest.mark.parametrize("name", list(GRIDS))
def test_residual_both_paths(name, odd):
    from paper_2004_13887_amd import dsw
    w = I.Workload(name, GRIDS[name], mach=1e-2, amplitude=0.5, steps=1, K=1, seed=601)
    print(f"[residual paths] {name} odd={odd}", flush=True)
    U0, tau = I.initial_state(w)
    Uk = I.random_fields(w.grid, 602, base=U0, scale=1e-3)
    R_o, Ub_o = oracle.residual(oracle.Grid(*w.grid.args()), oracle.Material(*w.material.astuple()), U0, Uk, tau)

    def place(a):
        t = torch.empty(a.size + odd, dtype=torch.float64, device="cuda")[odd:].view(a.shape)
        t.copy_(torch.as_tensor(a))
        return t

    gg = dsw.Grid.from_spec(w.grid, w.material)
    R, Ub = ({k: place(np.full(v.shape, 7.0)) for k, v in U0.items()} for _ in range(2))
    gg.residual({k: place(v) for k, v in U0.items()}, {k: place(v) for k, v in Uk.items()}, tau, R, Ub)
    torch.cuda.synchronize()
    gg.get_status()
    assert max(residual_errors(name, dsw.to_host(R), R_o, tau, w).values()) <= 1e-11
    for k, v in dsw.to_host(Ub).items():
        assert np.array_equal(v, Ub_o[k]), k


@pytest.mark.parametrize("form", ["plain", "pert", "forced"])
@pytest.mark.parametrize("nt", [120, 360])
def test_shell_forms(nt, form):
    """the residual's boundary shell with a workgroup per kind of row (120
    theta rows) and with one for all of them (360): one step, K = 1"""
    from helpers import random_wall
    from paper_2004_13887_amd import dsw
    spec = I.sector(3, nt, 200, 4e-4, 5e-4)
    w = I.Workload("shell", spec, mach=1e-2, amplitude=0.5, steps=1, K=1, seed=611)
    print(f"[shell] {spec.nr}x{nt}x{spec.np} {form}", flush=True)
    U0, tau = I.initial_state(w)
    og, om = oracle.Grid(*spec.args()), oracle.Material(*w.material.astuple())
    gg = dsw.Grid.from_spec(spec, w.material)
    out = gg.empty()
    if form == "plain":
        ref = oracle.split_step(og, om, U0, tau, 1)
        gg.split_step(dsw.to_device(U0), out, tau, 1)
    elif form == "pert":
        pbar, Tbar = I.reference_column(spec, w.material, I.T0)
        U0["p"] = np.ascontiguousarray(U0["p"] - pbar[:, None, None] + I.random_fields(spec, 612)["p"])
        ref = oracle.split_step_pert(og, om, U0, pbar, Tbar, tau, 1)
        gg.set_reference(pbar, Tbar)
        gg.split_step_pert(dsw.to_device(U0), out, tau, 1)
    else:
        wall, src = random_wall(spec, 613, scale=3.0), I.random_fields(spec, 614)
        ref = oracle.split_step(og, om, U0, tau, 1, wall0=wall, wall1=wall, src=src)
        gg.split_step_forced(dsw.to_device(U0), out, tau, 1, src=dsw.to_device(src), wall0=dsw.to_device(wall),
                             wall1=dsw.to_device(wall))
    torch.cuda.synchronize()
    gg.get_status()
    h = dsw.to_host(out)
    for k in h:
        e = np.linalg.norm(h[k] - ref[k]) / np.linalg.norm(ref[k])
        print(f"[shell] {form} {k}: {e:.2e}", flush=True)
        assert e <= 1e-11, k

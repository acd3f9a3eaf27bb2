"""Line passes at the sizes where they take two launches (block lines, then
scalar lines): the plain step with circles of uneven chunks, the perturbation
form, and the forced step with every forcing input, in r and theta lines of more
and of fewer than 128 rows (scalar lines in workgroups of 512 and of 256
threads), sector and sphere; the forced step's two-ended r and theta lines with
the scalar lines apart (512 rows), and its walked residual on a sphere.  Every
grid's launch counts are checked against the thresholds.  Bar: the parity tests'
1e-11 relative L2 per field against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import routes
from gpu_common import compare
from helpers import random_state, random_wall
from paper_2004_13887_amd import inputs as I

pytestmark = pytest.mark.gpu

FIELDS = ("p", "ur", "ut", "uf", "T")


def _spec(nr, nt, np_, sphere):
    return I.full_sphere(nr, nt, np_) if sphere else I.sector(nr, nt, np_, 4e-4, 5e-4)


def _assert_split(nr, nt, np_, sphere):
    assert routes.phi_lanes(nr, nt, np_, sphere) >= 2 ** 19
    assert min(routes.rt_workgroups(d, nr, nt, np_, sphere) for d in (0, 1)) >= 1024


@pytest.mark.parametrize("nr,nt,np_", [(128, 70, 90), (70, 136, 90)])
def test_uneven_circles(nr, nt, np_):
    from paper_2004_13887_amd import dsw
    _assert_split(nr, nt, np_, True)
    w = I.Workload("split", _spec(nr, nt, np_, True), mach=1e-3, amplitude=0.5, steps=1, K=1, seed=840 + nr)
    print(f"[split] {nr}x{nt}x{np_}", flush=True)
    U0, tau = I.initial_state(w)
    og, om = oracle.Grid(*w.grid.args()), oracle.Material(*w.material.astuple())
    gg = dsw.Grid.from_spec(w.grid, w.material)
    out, z, x = gg.empty(), gg.empty(), gg.empty()
    rhs, y = I.random_fields(w.grid, 31), I.random_fields(w.grid, 32)
    gg.split_step(dsw.to_device(U0), out, tau, 1)
    gg.line_solve(2, dsw.to_device(U0), tau, dsw.to_device(rhs), x)
    gg.line_solve_T(2, dsw.to_device(U0), tau, dsw.to_device(y), z)
    torch.cuda.synchronize()
    gg.get_status()
    e = compare("step", dsw.to_host(out), oracle.split_step(og, om, U0, tau, 1), base=U0)
    assert max(e[k] for k in FIELDS) <= 1e-11
    hx, hz = dsw.to_host(x), dsw.to_host(z)
    lhs = sum(float(np.vdot(hz[k], rhs[k])) for k in FIELDS)
    both = sum(float(np.vdot(y[k], hx[k])) for k in FIELDS)
    size = sum(float(np.linalg.norm(y[k]) * np.linalg.norm(hx[k])) for k in FIELDS)
    assert abs(lhs - both) <= 1e-10 * size  # the adjoint tests' bar


@pytest.mark.parametrize("nr,nt,np_,sphere", [(136, 128, 64, True), (128, 136, 62, False), (120, 150, 64, False)])
def test_perturbation_step(nr, nt, np_, sphere):
    from paper_2004_13887_amd import dsw
    _assert_split(nr, nt, np_, sphere)
    w = I.Workload("split", _spec(nr, nt, np_, sphere), mach=1e-3, amplitude=0.5, steps=1, K=1, seed=850 + nr)
    print(f"[split pert] {nr}x{nt}x{np_} sphere={sphere}", flush=True)
    U0, tau = I.initial_state(w)
    pbar, Tbar = I.reference_column(w.grid, w.material, I.T0)
    U0["p"] = np.ascontiguousarray(U0["p"] - pbar[:, None, None] + I.random_fields(w.grid, 852)["p"])
    ref = oracle.split_step_pert(oracle.Grid(*w.grid.args()), oracle.Material(*w.material.astuple()), U0, pbar, Tbar,
                                 tau, 1)
    gg = dsw.Grid.from_spec(w.grid, w.material)
    gg.set_reference(pbar, Tbar)
    out = gg.empty()
    gg.split_step_pert(dsw.to_device(U0), out, tau, 1)
    torch.cuda.synchronize()
    gg.get_status()
    e = compare("split pert", dsw.to_host(out), ref, base=U0)
    assert max(e[k] for k in FIELDS) <= 1e-11


FORCED = [(70, 136, 130, False, "split"), (136, 128, 64, True, "split"), (512, 4, 5, False, "apart"),
          (4, 512, 5, False, "apart"), (512, 3, 8, True, "apart"), (20, 67, 256, True, "walk"),
          (9, 147, 256, True, "walk")]


@pytest.mark.parametrize("nr,nt,np_,sphere,route", FORCED)
def test_forced_step(nr, nt, np_, sphere, route):
    from paper_2004_13887_amd import dsw
    if route == "split":
        _assert_split(nr, nt, np_, sphere)
    elif route == "walk":
        assert routes.march_workgroups(nr, nt, np_) >= 450
    else:
        assert max(nr, nt) > 256 and max(nr, nt) % 8 == 0 and 256 % (max(nr, nt) // 8) == 0
    spec = _spec(nr, nt, np_, sphere)
    print(f"[split forced] {nr}x{nt}x{np_} sphere={sphere} {route}", flush=True)
    U0, tau = random_state(spec, 861, mach=0.05)
    rng = np.random.Generator(np.random.PCG64(862))
    scale = {"p": 1e-4 * np.mean(U0["p"]), "ur": 1.0, "ut": 1.0, "uf": 1.0, "T": 1e-3 * np.mean(U0["T"])}
    src = {k: scale[k] * rng.uniform(-1.0, 1.0, v.shape) for k, v in U0.items()}
    bnd = {k: U0[k] + rng.uniform(-2.0, 2.0, U0[k].shape) for k in ("ur", "ut", "uf")}
    full = dict(bnd, p=U0["p"], T=U0["T"])
    w0, w1 = random_wall(spec, 863, scale=3.0), random_wall(spec, 864, scale=3.0)
    ref = oracle.split_step(oracle.Grid(*spec.args()), oracle.Material(*I.AIR.astuple()), U0, tau, 2, wall0=w0,
                            wall1=w1, src=src, bnd=full)
    gg = dsw.Grid.from_spec(spec, I.AIR)
    out = gg.empty()
    gg.split_step_forced(dsw.to_device(U0), out, tau, 2, src=dsw.to_device(src), wall0=dsw.to_device(w0),
                         wall1=dsw.to_device(w1), bnd=dsw.to_device(full))
    torch.cuda.synchronize()
    gg.get_status()
    e = compare("split forced", dsw.to_host(out), ref, base=U0)
    assert max(e[k] for k in FIELDS) <= 1e-11

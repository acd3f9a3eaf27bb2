"""The residual of large grids, whose interior is walked plane by plane through
a window in LDS, at the edges of its tiles: phi lines a tile wide and one off
it, theta tiles and r segments that the grid does not fill, segments of two and
of four planes, the smallest grid that takes it (450 workgroups of two planes)
and one below, the shell in the same launch and in one of its own.  Bar: the
parity tests' 1e-11 relative L2 per field against the oracle; a batch gives
bitwise the states of single steps."""
import numpy as np
import pytest
import torch

import oracle
from paper_2004_13887_amd import inputs as I
from test_gpu_parity import residual_errors

pytestmark = pytest.mark.gpu

SIZES = [(19, 66, 260), (20, 67, 321), (35, 130, 63), (36, 129, 64), (8, 146, 256), (5, 601, 65), (27, 141, 65),
         (4, 700, 129)]


def _workload(nr, nt, np_, sphere, K):
    spec = I.full_sphere(nr, nt, np_) if sphere else I.sector(nr, nt, np_, 4e-4, 5e-4)
    return I.Workload("march", spec, mach=1e-2, amplitude=0.5, steps=1, K=K, seed=700 + nr)


@pytest.mark.parametrize("sphere", [False, True])
@pytest.mark.parametrize("nr,nt,np_", SIZES)
def test_tile_edges(nr, nt, np_, sphere):
    from paper_2004_13887_amd import dsw
    w = _workload(nr, nt, np_, sphere, 1)
    print(f"[march] {nr}x{nt}x{np_} sphere={sphere}", flush=True)
    U0, tau = I.initial_state(w)
    Uk = I.random_fields(w.grid, 702, base=U0, scale=1e-3)
    R_o, _ = oracle.residual(oracle.Grid(*w.grid.args()), oracle.Material(*w.material.astuple()), U0, Uk, tau)
    gg = dsw.Grid.from_spec(w.grid, w.material)
    R, Ub = gg.empty(), gg.empty()
    for v in R.values():
        v.fill_(7.0)
    gg.residual(dsw.to_device(U0), dsw.to_device(Uk), tau, R, Ub)
    torch.cuda.synchronize()
    gg.get_status()
    assert max(residual_errors("march", dsw.to_host(R), R_o, tau, w).values()) <= 1e-11


@pytest.mark.parametrize("nr,nt,np_", [(19, 66, 260), (36, 129, 64)])
def test_perturbation_form(nr, nt, np_):
    from paper_2004_13887_amd import dsw
    w = _workload(nr, nt, np_, False, 2)
    print(f"[march pert] {nr}x{nt}x{np_}", flush=True)
    U0, tau = I.initial_state(w)
    og, om = oracle.Grid(*w.grid.args()), oracle.Material(*w.material.astuple())
    pbar, Tbar = I.reference_column(w.grid, w.material, I.T0)
    U0["p"] = np.ascontiguousarray(U0["p"] - pbar[:, None, None] + I.random_fields(w.grid, 712)["p"])
    ref = oracle.split_step_pert(og, om, U0, pbar, Tbar, tau, w.K)
    gg = dsw.Grid.from_spec(w.grid, w.material)
    out = gg.empty()
    gg.set_reference(pbar, Tbar)
    gg.split_step_pert(dsw.to_device(U0), out, tau, w.K)
    torch.cuda.synchronize()
    gg.get_status()
    h = dsw.to_host(out)
    for k in h:
        assert np.linalg.norm(h[k] - ref[k]) <= 1e-11 * np.linalg.norm(ref[k]), k


def test_batch_is_bitwise_the_single_steps():
    from paper_2004_13887_amd import dsw
    ws = [_workload(*s) for s in [(19, 66, 260, False, 2), (35, 130, 63, False, 2), (5, 7, 9, False, 2),
                                  (19, 66, 256, True, 2)]]
    print("[march batch]", flush=True)
    E = dsw.Ensemble([w.grid for w in ws], [w.material for w in ws])
    states = [I.initial_state(w) for w in ws]
    U = [dsw.to_device(s[0]) for s in states]
    out = [g.empty() for g in E.members]
    E.ensemble_step(U, out, [s[1] for s in states], 2)
    for g, u, s, o in zip(E.members, U, states, out):
        one = g.empty()
        g.split_step(u, one, s[1], 2)
        torch.cuda.synchronize()
        g.get_status()
        assert all(torch.equal(o[k], one[k]) for k in o)


@pytest.mark.parametrize("nr,nt,np_", [(19, 66, 260), (36, 129, 64), (4, 700, 129)])
def test_forced_form(nr, nt, np_):
    from helpers import random_wall
    from paper_2004_13887_amd import dsw
    w = _workload(nr, nt, np_, False, 1)
    print(f"[march forced] {nr}x{nt}x{np_}", flush=True)
    U0, tau = I.initial_state(w)
    og, om = oracle.Grid(*w.grid.args()), oracle.Material(*w.material.astuple())
    gg = dsw.Grid.from_spec(w.grid, w.material)
    full, src = random_wall(w.grid, 721, scale=3.0), I.random_fields(w.grid, 722)
    part = {k: v for k, v in full.items() if k in ("ur_p1", "ut_p2", "uf_r1")}  # the rest absent: zero
    for wall in (full, part):
        out = gg.empty()
        ref = oracle.split_step(og, om, U0, tau, 1, wall0=wall, wall1=wall, src=src)
        gg.split_step_forced(dsw.to_device(U0), out, tau, 1, src=dsw.to_device(src), wall0=dsw.to_device(wall),
                             wall1=dsw.to_device(wall))
        torch.cuda.synchronize()
        gg.get_status()
        h = dsw.to_host(out)
        for k in h:
            assert np.linalg.norm(h[k] - ref[k]) <= 1e-11 * np.linalg.norm(ref[k]), k


@pytest.mark.parametrize("form", ["plain", "pert", "forced"])
def test_more_rows_than_one_launch_numbers(form):
    """a grid whose shell does not fit the interior's launch (its third
    dimension holds 65535 workgroups): every point by the general rules"""
    from helpers import random_wall
    from paper_2004_13887_amd import dsw
    w = _workload(6000, 3, 4, False, 1)
    print(f"[rows] 6000x3x4 {form}", flush=True)
    U0, tau = I.initial_state(w)
    og, om = oracle.Grid(*w.grid.args()), oracle.Material(*w.material.astuple())
    gg = dsw.Grid.from_spec(w.grid, w.material)
    out = gg.empty()
    if form == "plain":
        ref = oracle.split_step(og, om, U0, tau, 1)
        gg.split_step(dsw.to_device(U0), out, tau, 1)
    elif form == "pert":
        pbar, Tbar = I.reference_column(w.grid, w.material, I.T0)
        U0["p"] = np.ascontiguousarray(U0["p"] - pbar[:, None, None] + I.random_fields(w.grid, 732)["p"])
        ref = oracle.split_step_pert(og, om, U0, pbar, Tbar, tau, 1)
        gg.set_reference(pbar, Tbar)
        gg.split_step_pert(dsw.to_device(U0), out, tau, 1)
    else:
        wall, src = random_wall(w.grid, 733, scale=3.0), I.random_fields(w.grid, 734)
        ref = oracle.split_step(og, om, U0, tau, 1, wall0=wall, wall1=wall, src=src)
        gg.split_step_forced(dsw.to_device(U0), out, tau, 1, src=dsw.to_device(src), wall0=dsw.to_device(wall),
                             wall1=dsw.to_device(wall))
    torch.cuda.synchronize()
    gg.get_status()
    h = dsw.to_host(out)
    for k in h:
        assert np.linalg.norm(h[k] - ref[k]) <= 1e-11 * np.linalg.norm(ref[k]), k

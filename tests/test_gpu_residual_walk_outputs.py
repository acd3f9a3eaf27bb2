"""What the walked residual writes beside R: the midpoint, at every entry of the
tile-edge grids of test_gpu_residual_march.py (bitwise the oracle's, over a
sentinel), also where the caller's arrays start at an odd multiple of 8 bytes;
and the status words, for a value planted in the walked interior, at its tile
and segment edges and in the shell, by every form of it (step, C-ABI call,
perturbation form, forced, batch)."""
import math

import numpy as np
import pytest
import torch

import oracle
import routes
import test_gpu_residual_march as march
from paper_2004_13887_amd import inputs as I

pytestmark = pytest.mark.gpu


def _odd(fields, fill=None):
    """the same fields in arrays that start 8 bytes past a 16-byte boundary"""
    out = {}
    for k, v in fields.items():
        buf = torch.empty(v.numel() + 3, dtype=torch.float64, device="cuda")
        at = 1 if buf.data_ptr() % 16 == 0 else 0
        out[k] = buf[at:at + v.numel()].view(v.shape)
        assert out[k].data_ptr() % 16 == 8
        if fill is None:
            out[k].copy_(v)
        else:
            out[k].fill_(fill)
    return out


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("sphere", [False, True])
@pytest.mark.parametrize("nr,nt,np_", march.SIZES)
def test_midpoint_written_everywhere(nr, nt, np_, sphere, odd):
    from paper_2004_13887_amd import dsw
    w = march._workload(nr, nt, np_, sphere, 1)
    print(f"[walk midpoint] {nr}x{nt}x{np_} sphere={sphere} odd={odd}", flush=True)
    U0, tau = I.initial_state(w)
    Uk = I.random_fields(w.grid, 703, base=U0, scale=1e-3)
    R_o, Ub_o = oracle.residual(oracle.Grid(*w.grid.args()), oracle.Material(*w.material.astuple()), U0, Uk, tau)
    gg = dsw.Grid.from_spec(w.grid, w.material)
    dU, dk = dsw.to_device(U0), dsw.to_device(Uk)
    R, Ub = gg.empty(), gg.empty()
    if odd:
        dU, dk, R, Ub = _odd(dU), _odd(dk), _odd(R, 7.0), _odd(Ub, 7.0)
    else:
        for v in list(R.values()) + list(Ub.values()):
            v.fill_(7.0)
    gg.residual(dU, dk, tau, R, Ub)
    torch.cuda.synchronize()
    gg.get_status()
    for k, v in dsw.to_host(Ub).items():
        assert np.array_equal(v, Ub_o[k]), k
    errs = march.residual_errors("walk", dsw.to_host(R), R_o, tau, w)
    assert max(errs.values()) <= 1e-11


NR, NT, NP = 19, 66, 260
PLANTS = [("T", (9, 33, 100), -1.0, "DSW_ENONPHYS"), ("T", (1, 1, 0), -1.0, "DSW_ENONPHYS"),
          ("T", (17, 64, 259), 0.0, "DSW_ENONPHYS"), ("T", (0, 33, 63), -1.0, "DSW_ENONPHYS"),
          ("T", (5, 65, 64), -1.0, "DSW_ENONPHYS"), ("ur", (9, 33, 100), math.nan, "DSW_EDIVERGED"),
          ("uf", (17, 64, 259), math.inf, "DSW_EDIVERGED"), ("ut", (2, 2, 63), math.nan, "DSW_EDIVERGED"),
          ("p", (16, 61, 64), math.nan, "DSW_EDIVERGED"), ("p", (18, 65, 259), math.nan, "DSW_EDIVERGED")]


@pytest.mark.parametrize("form", ["step", "call", "pert", "forced", "batch"])
@pytest.mark.parametrize("field,index,value,code", PLANTS)
def test_status_of_a_planted_value(field, index, value, code, form):
    from paper_2004_13887_amd import dsw
    assert routes.march_workgroups(NR, NT, NP) >= 450
    w = march._workload(NR, NT, NP, False, 1)
    print(f"[walk status] {form} {field}{index} = {value} -> {code}", flush=True)
    clean, tau = I.initial_state(w)
    pbar, Tbar = I.reference_column(w.grid, w.material, I.T0)
    if form == "pert":
        clean["p"] = np.ascontiguousarray(clean["p"] - pbar[:, None, None])
    bad = {k: v.copy() for k, v in clean.items()}
    bad[field][index] = value
    if form == "batch":
        other = march._workload(5, 7, 9, False, 1)
        E = dsw.Ensemble([other.grid, w.grid], [other.material, w.material])
        dO, tau_o = dsw.to_device(I.initial_state(other)[0]), I.initial_state(other)[1]
        out = [g.empty() for g in E.members]
    else:
        gg = dsw.Grid.from_spec(w.grid, w.material)
        out, Ub = gg.empty(), gg.empty()
        if form == "pert":
            gg.set_reference(pbar, Tbar)
    for U, expect in ((bad, getattr(dsw, code)), (clean, dsw.DSW_OK)):
        dU = dsw.to_device(U)
        if form == "batch":
            E.ensemble_step([dO, dU], out, [tau_o, tau], 1)
        elif form == "step":
            gg.split_step(dU, out, tau, 1)
        elif form == "call":
            gg.residual(dU, dU, tau, out, Ub)
        elif form == "pert":
            gg.split_step_pert(dU, out, tau, 1)
        else:
            gg.split_step_forced(dU, out, tau, 1)
        torch.cuda.synchronize()
        status = E.get_status if form == "batch" else gg.get_status
        if expect == dsw.DSW_OK:
            assert status() == dsw.DSW_OK  # read and cleared
        else:
            with pytest.raises(dsw.DswError) as ei:
                status()
            assert ei.value.code == expect, str(ei.value)

"""The partitioned r and theta solvers at the edges of their chunks: lines one
row off a multiple of the rows per chunk (fillers at the head of the first
chunk), a single chunk, the longest line the default takes and the first it
does not, workgroups that the lines do not fill, lanes whose lines straddle the
phi ends of a plane, poles and walls.  Bars: the parity tests' 1e-11 relative
L2 per field against the oracle; for the transposed systems, which take the
same chunks, the adjoint tests' 1e-10 on <M^-T y, b> = <y, M^-1 b>."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import compare
from paper_2004_13887_amd import inputs as I

pytestmark = pytest.mark.gpu

SIZES = [(3, 4, 3), (5, 3, 4), (8, 9, 5), (7, 12, 65), (17, 33, 6), (64, 5, 9), (129, 3, 7), (3, 130, 5), (200, 4, 7),
         (4, 201, 3), (255, 3, 4), (3, 256, 11), (257, 3, 3), (3, 259, 4)]


@pytest.mark.parametrize("sphere", [False, True])
@pytest.mark.parametrize("nr,nt,np_", SIZES)
def test_chunk_edges(nr, nt, np_, sphere):
    from paper_2004_13887_amd import dsw
    spec = I.full_sphere(nr, nt, np_) if sphere else I.sector(nr, nt, np_, 4e-4, 5e-4)
    w = I.Workload("edges", spec, mach=1e-2, amplitude=0.5, steps=1, K=1, seed=800 + nr + nt)
    print(f"[rt chunks] {nr}x{nt}x{np_} sphere={sphere}", flush=True)
    U0, tau = I.initial_state(w)
    og, om = oracle.Grid(*spec.args()), oracle.Material(*w.material.astuple())
    gg = dsw.Grid.from_spec(spec, w.material)
    dU0 = dsw.to_device(U0)
    for d in (0, 1):
        rhs = I.random_fields(spec, 41 + d)
        ref = oracle.line_solve(og, om, U0, tau, d, rhs)
        for bs in (64, 256):  # workgroups of few and of many lines
            gg.set_config(sweep_block_r=bs, sweep_block_theta=bs)
            x = gg.empty()
            for v in x.values():
                v.fill_(7.0)
            gg.line_solve(d, dU0, tau, dsw.to_device(rhs), x)
            torch.cuda.synchronize()
            gg.get_status()
            e = compare(f"d={d} bs={bs}", dsw.to_host(x), ref)
            assert max(e.values()) <= 1e-11
            hx = dsw.to_host(x)
            for k in ("ur", "ut"):  # boundary-normal faces are zero
                faces = (hx[k][0], hx[k][-1]) if k == "ur" else (hx[k][:, 0], hx[k][:, -1])
                assert not np.any(faces[0]) and not np.any(faces[1])
            y = I.random_fields(spec, 51 + d)
            gg.line_solve_T(d, dU0, tau, dsw.to_device(y), x)
            torch.cuda.synchronize()
            gg.get_status()
            hz = dsw.to_host(x)
            lhs = sum(float(np.vdot(hz[k], rhs[k])) for k in hx)
            both = sum(float(np.vdot(y[k], hx[k])) for k in hx)
            size = sum(float(np.linalg.norm(y[k]) * np.linalg.norm(hx[k])) for k in hx)
            assert abs(lhs - both) <= 1e-10 * size, (d, bs)

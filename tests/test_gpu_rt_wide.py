"""Scalar r and theta lines of more than 128 rows, whose launches take 512
threads per workgroup: beside partitioned block lines (lines of 17 chunks that
do not fill a workgroup, sector and sphere) and beside two-ended ones (512
rows).  Bars: the parity tests' 1e-11 relative L2 per field against the
oracle; for the transposed systems the adjoint tests' 1e-10 on
<M^-T y, b> = <y, M^-1 b>."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import compare
from paper_2004_13887_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,nr,nt,np_,sphere", [(0, 136, 9, 801, False), (1, 9, 136, 801, False),
                                                (1, 9, 131, 803, True), (0, 512, 4, 5, False), (1, 4, 512, 5, True)])
def test_wide_scalar_lines(d, nr, nt, np_, sphere):
    from paper_2004_13887_amd import dsw
    spec = I.full_sphere(nr, nt, np_) if sphere else I.sector(nr, nt, np_, 4e-4, 5e-4)
    w = I.Workload("wide", spec, mach=1e-2, amplitude=0.5, steps=1, K=1, seed=820 + nr + nt)
    print(f"[rt wide] d={d} {nr}x{nt}x{np_} sphere={sphere}", flush=True)
    U0, tau = I.initial_state(w)
    og, om = oracle.Grid(*spec.args()), oracle.Material(*w.material.astuple())
    gg = dsw.Grid.from_spec(spec, w.material)
    dU0 = dsw.to_device(U0)
    rhs, y = I.random_fields(spec, 41 + d), I.random_fields(spec, 51 + d)
    x, z = gg.empty(), gg.empty()
    gg.line_solve(d, dU0, tau, dsw.to_device(rhs), x)
    gg.line_solve_T(d, dU0, tau, dsw.to_device(y), z)
    torch.cuda.synchronize()
    gg.get_status()
    hx, hz = dsw.to_host(x), dsw.to_host(z)
    e = compare(f"d={d}", hx, oracle.line_solve(og, om, U0, tau, d, rhs))
    assert max(e.values()) <= 1e-11
    lhs = sum(float(np.vdot(hz[k], rhs[k])) for k in hx)
    both = sum(float(np.vdot(y[k], hx[k])) for k in hx)
    size = sum(float(np.linalg.norm(y[k]) * np.linalg.norm(hx[k])) for k in hx)
    assert abs(lhs - both) <= 1e-10 * size

"""The fused reverse of the local rows at the edges of its tiles: circles and
regions a full tile wide, one off it and several tiles wide (first tiles in
which no lane is a ghost), segments and theta tiles that the grid does not
fill, the smallest grids, poles and walls.  Bar: the adjoint tests'
1e-10 on <J^T lam, v> = <lam, J v> against the complex-step oracle, relative
to the sum of the fields' contributions."""
import numpy as np
import pytest
import torch

import oracle
from paper_2004_13887_amd import inputs as I

pytestmark = pytest.mark.gpu

SCALE = {"p": 1.0, "ur": 1e-2, "ut": 1e-2, "uf": 1e-2, "T": 1e-2}
SIZES = [(3, 3, 64), (4, 5, 65), (6, 7, 130), (11, 12, 66), (10, 14, 128), (12, 11, 192), (3, 5, 63), (5, 3, 67),
         (19, 3, 5), (3, 20, 4)]


@pytest.mark.parametrize("sphere", [False, True])
@pytest.mark.parametrize("nr,nt,np_", SIZES)
def test_tile_edges(nr, nt, np_, sphere):
    from paper_2004_13887_amd import dsw
    spec = I.full_sphere(nr, nt, np_) if sphere else I.sector(nr, nt, np_, 4e-4, 5e-4)
    w = I.Workload("tiles", spec, mach=1e-2, amplitude=0.5, steps=1, K=2, seed=900 + nr + nt)
    print(f"[adjoint tiles] {nr}x{nt}x{np_} sphere={sphere}", flush=True)
    U0, tau = I.initial_state(w)
    og, om = oracle.Grid(*spec.args()), oracle.Material(*w.material.astuple())
    gg = dsw.Grid.from_spec(spec, w.material)
    rng = np.random.Generator(np.random.PCG64(91))
    lam = {k: rng.uniform(-1.0, 1.0, s) / SCALE[k] for k, s in spec.shapes().items()}
    V = {k: SCALE[k] * rng.uniform(-1.0, 1.0, s) for k, s in spec.shapes().items()}
    _, dU1 = oracle.jvp_split_step(og, om, U0, V, tau, w.K)
    out = gg.empty()
    gg.adjoint_step(dsw.to_device(U0), tau, w.K, dsw.to_device(lam), out)
    torch.cuda.synchronize()
    gg.get_status()
    got = dsw.to_host(out)
    lhs = {k: float(np.vdot(got[k], V[k])) for k in V}
    rhs = {k: float(np.vdot(lam[k], dU1[k])) for k in V}
    size = sum(abs(v) for v in lhs.values()) + sum(abs(v) for v in rhs.values())
    assert abs(sum(lhs.values()) - sum(rhs.values())) <= 1e-10 * size

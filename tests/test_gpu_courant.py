"""The Courant numbers' maxima wherever they sit: the peak velocity and the
peak temperature at the first and last cell of every direction, on rows shorter
and longer than a wave, more rows than one launch holds waves, and T <= 0 or a
NaN ignored as the oracle's comparisons ignore them.  The kernel evaluates the
oracle's expressions, so the bar is the parity test's 1e-14."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2004_13887_amd import inputs as I

pytestmark = pytest.mark.gpu

GRIDS = [I.sector(3, 3, 3, 0.01, 0.01), I.sector(5, 7, 63, 1e-3, 1e-3), I.full_sphere(4, 6, 64),
         I.full_sphere(3, 5, 65), I.sector(100, 101, 130, 1e-4, 1e-4)]


@pytest.mark.parametrize("spec", GRIDS, ids=lambda g: f"{g.nr}x{g.nt}x{g.np}")
@pytest.mark.parametrize("where", [0, -1])
def test_maxima_anywhere(spec, where):
    from paper_2004_13887_amd import dsw
    rng = np.random.Generator(np.random.PCG64(701))
    U = {k: np.ascontiguousarray(rng.uniform(-1.0, 1.0, s)) for k, s in spec.shapes().items()}
    U["T"] = np.ascontiguousarray(300.0 + U["T"])
    U["uf"][where, where, where] = 50.0
    U["T"][where, where, where] = 400.0
    U["T"].flat[U["T"].size // 2] = -5.0
    U["ur"].flat[U["ur"].size // 2] = np.nan
    og, om = oracle.Grid(*spec.args()), oracle.Material(*I.AIR.astuple())
    gg = dsw.Grid.from_spec(spec, I.AIR)
    dU = dsw.to_device(U)
    for tau in (0.3, 2.0):  # a second call starts from cleared maxima
        ref, got = oracle.courant(og, om, U, tau), gg.courant(dU, tau)
        print(f"[courant] {spec.nr}x{spec.nt}x{spec.np} at {where}: {got} oracle {ref}", flush=True)
        for a, b in zip(got, ref):
            assert math.isclose(a, b, rel_tol=1e-14)

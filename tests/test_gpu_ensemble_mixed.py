"""A batch whose members take different solvers in the same pass, in r, theta
and phi: lines of 512 rows (two-ended, the scalar lines apart in workgroups of
512 threads), of 264 (two-ended in one launch: 33 chunks of 8 do not divide a
workgroup), of 64 (partitioned); a circle of 1028 cells (one thread per line)
beside partitioned circles and sectors.  Each member's solver is checked on its
own line solves (bitwise those of the solver named explicitly), then the
batched step: bitwise the members' own steps, and against the oracle."""
import math

import pytest
import torch

import oracle
from gpu_common import compare
from paper_2004_13887_amd import inputs as I

pytestmark = pytest.mark.gpu

K = 2
FIELDS = ("p", "ur", "ut", "uf", "T")


def _sec(nr, nt, np_, seed):
    return I.Workload(f"sec{seed}", I.sector(nr, nt, np_, math.radians(20) / nt, math.radians(24) / np_), mach=1e-2,
                      amplitude=0.5, steps=1, K=K, seed=seed)


def _sph(nr, nt, np_, seed):
    return I.Workload(f"sph{seed}", I.full_sphere(nr, nt, np_), mach=1e-3, amplitude=0.5, steps=1, K=K, seed=seed)


# direction, members, rows per thread that each takes (0: two-ended / thread per line)
BATCHES = [(1, [_sec(4, 512, 6, 331), _sec(4, 264, 8, 332), _sec(5, 64, 10, 333), _sph(3, 512, 8, 334)], [0, 0, 4, 0]),
           (0, [_sec(264, 4, 6, 335), _sec(512, 3, 8, 336), _sph(64, 5, 12, 337)], [0, 0, 4]),
           (2, [_sph(3, 4, 1028, 338), _sph(4, 5, 12, 339), _sec(3, 4, 1028, 340), _sec(5, 7, 9, 341)], [0, 4, 0, 4])]


@pytest.mark.parametrize("d,ws,rows", BATCHES, ids=["theta", "r", "phi"])
def test_members_with_different_solvers(d, ws, rows):
    from paper_2004_13887_amd import dsw
    print("[ensemble mixed]", d, [(w.grid.nr, w.grid.nt, w.grid.np) for w in ws], flush=True)
    E = dsw.Ensemble([w.grid for w in ws], [w.material for w in ws])
    states = [I.initial_state(w) for w in ws]
    U, taus = [dsw.to_device(s[0]) for s in states], [s[1] for s in states]
    out = [g.empty() for g in E.members]
    E.ensemble_step(U, out, taus, K)
    torch.cuda.synchronize()
    E.get_status()
    key = {0: ("rows_per_thread_r", -1), 1: ("rows_per_thread_theta", -1), 2: ("phi_rows_per_thread", 4)}[d]
    for w, g, u, s, o, pm in zip(ws, E.members, U, states, out, rows):
        one = g.empty()
        g.split_step(u, one, s[1], K)
        grid = dsw.Grid.from_spec(w.grid, w.material)
        rhs, x = dsw.to_device(I.random_fields(w.grid, 41 + d)), {}
        for q in (key[1], 0) if d == 2 else (key[1], 0, 4):
            grid.set_config(**{key[0]: q})
            x[q] = grid.empty()
            grid.line_solve(d, u, s[1], rhs, x[q])
        torch.cuda.synchronize()
        g.get_status()
        line = all(torch.equal(x[key[1]][k], x[0][k]) for k in FIELDS)
        assert line == (pm == 0), (w.name, "takes the other solver")
        assert all(torch.equal(o[k], one[k]) for k in FIELDS), w.name
        ref = oracle.split_step(oracle.Grid(*w.grid.args()), oracle.Material(*w.material.astuple()), s[0], s[1], K)
        e = compare(w.name, dsw.to_host(o), ref, base=s[0])
        assert max(e[k] for k in FIELDS) <= 1e-11

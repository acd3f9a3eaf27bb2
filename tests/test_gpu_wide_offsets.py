"""Line solves of grids whose arrays reach 4 GiB, where the partitioned solvers
take 64-bit byte offsets: the lines at the first and last 64 phi cells (r planes)
are bitwise those of a grid of these cells alone, whose spacings and metric
factors are the same numbers (powers of two), and which takes 32-bit offsets.
Lines that read a neighbour beyond the cut are left out."""
import pytest
import torch

from paper_2004_13887_amd import inputs as I

pytestmark = pytest.mark.gpu

H = 2.0 ** -20
TAU = 1e-7
N = 2 ** 19 + 5  # times 1024: 5120 cells past 4 GiB of doubles


def _state(grid, periodic, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    U = grid.empty()
    lo = {"p": (9.9e4, 1.01e5), "T": (299.0, 301.0)}
    for k, v in U.items():
        v.uniform_(*lo.get(k, (-1.0, 1.0)), generator=g)
    for f in (U["ur"][0], U["ur"][-1], U["ut"][:, 0], U["ut"][:, -1]):
        f.zero_()
    if not periodic:
        U["uf"][:, :, 0].zero_()
        U["uf"][:, :, -1].zero_()
    return U


def _cut(U, axis, at, n):
    """the cells [at, at + n) along axis and the faces around them, the outer
    ones the walls of a grid of their own"""
    own = {0: "ur", 2: "uf"}[axis]
    V = {k: v.narrow(axis, at, n + (1 if k == own else 0)).clone() for k, v in U.items()}
    V[own].narrow(axis, 0, 1).zero_()
    V[own].narrow(axis, n, 1).zero_()
    return V


@pytest.mark.parametrize("axis,periodic", [(2, False), (0, False), (0, True)])
def test_lines_past_4_gib(axis, periodic):
    from paper_2004_13887_amd import dsw
    torch.cuda.empty_cache()
    if axis == 2:  # r and theta lines of 32 rows, N phi cells
        make = lambda at, n: dsw.Grid(32, 32, n, 1.0, 1.25, 1.0, 1.25, at * H, (at + n) * H, 0, I.AIR.astuple())
        dirs = (0, 1)
    else:          # phi lines of 64 cells, N r planes
        p2 = 2.0 * torch.pi if periodic else 0.25
        make = lambda at, n: dsw.Grid(n, 16, 64, 1.0 + at * H, 1.0 + (at + n) * H, 1.0, 1.25, 0.0, p2,
                                      int(periodic), I.AIR.astuple())
        dirs = (2,)
    need = 1024 * N * 8 * (7 * 5.2 + 27)  # the workspace, two states and the sweep scratch
    free = torch.cuda.mem_get_info()[0]
    print(f"[wide] axis {axis} periodic={periodic}: {need / 2**30:.0f} of {free / 2**30:.0f} GiB", flush=True)
    if free < need:
        pytest.skip("the grid does not fit this GPU's free memory")
    big = make(0, N)
    small = []
    try:
        U, x = _state(big, periodic, 77), big.empty()
        for at in (0, N - 64):
            grid = make(at, 64)
            small.append((at, grid, _cut(U, axis, at, 64), grid.empty()))
        for d in dirs:
            for transposed in (False, True):
                solve = (lambda g, *a: g.line_solve_T(d, *a)) if transposed else (lambda g, *a: g.line_solve(d, *a))
                solve(big, U, TAU, U, x)
                torch.cuda.synchronize()
                big.get_status()
                for at, grid, V, y in small:
                    solve(grid, V, TAU, V, y)
                    torch.cuda.synchronize()
                    grid.get_status()
                    for k in y:
                        a, b = x[k].narrow(axis, at + 2, 60), y[k].narrow(axis, 2, 60)
                        assert torch.equal(a, b), (d, transposed, at, k, float((a - b).abs().max()))
    finally:
        big.free_grid()
        for _, grid, _, _ in small:
            grid.free_grid()
        U = x = small = None
        torch.cuda.empty_cache()

"""Launch counts that the tests of split launches check their grids against
(test infrastructure): the chunks, workgroups and lanes of the partitioned line
solvers at their default 256 threads and 4 rows per thread."""


def ceil(a, b):
    return -(-a // b)


def phi_lanes(nr, nt, np_, cyclic):
    """lanes of the phi pass; from 2**19 on its block and scalar lines take two launches"""
    T = ceil(np_, 4)
    if cyclic:
        T = 1 << (T - 1).bit_length()
    use = {bs: bs // T * T / bs for bs in (64, 128, 256)}
    bs = next((b for b in (64, 128) if use[b] >= 0.95 * max(use.values())), 256)
    return 2 * ceil(nr * nt, bs // T) * bs


def rt_workgroups(d, nr, nt, np_, cyclic):
    """workgroups of a partitioned r (0) or theta (1) pass; from 1024 on it takes two launches"""
    n, m = (nr, nt) if d == 0 else (nt, nr)
    L, L8 = 256 // ceil(n, 4), 256 // ceil(n, 8)
    return ceil(m * np_, L) + ceil((m - 1) * np_, L8) + ceil(m * (np_ - (0 if cyclic else 1)), L8)


def march_workgroups(nr, nt, np_):
    """workgroups of two planes of the walked residual, taken from 450 on"""
    return ceil(np_, 64) * ceil(nt - 2, 4) * ceil(nr - 2, 2)

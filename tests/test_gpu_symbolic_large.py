"""GPU symbolic phase on patterns of enough rows for the small tables: grids of
7 and 27 points and chains with hubs, whose rows fit and outgrow every table, and
level sets of long lists of rows and columns.  Integer work: equal to the oracle.
A search given up for a larger table costs a bounded part of the search, and
lists of columns no more than lists of rows."""
import time

import numpy as np
import pytest
import torch

from paper_1703_01325_amd import synth

from test_gpu_symbolic import api, check_vs_oracle, cuda_i32  # noqa: F401
from test_gpu_symbolic_tables import wide_row_pattern

pytestmark = pytest.mark.gpu


def _csr(rows, cols, nb):
    o = np.lexsort((cols, rows))
    rows, cols = rows[o], cols[o]
    return np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=nb))]).astype(np.int32), cols.astype(np.int32)


def stencil27_pattern(n):
    i = np.arange(n ** 3)
    x, y, z = i % n, i // n % n, i // n // n
    rows, cols = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                m = (x + dx >= 0) & (x + dx < n) & (y + dy >= 0) & (y + dy < n) & (z + dz >= 0) & (z + dz < n)
                rows.append(i[m])
                cols.append(i[m] + dx + n * (dy + n * dz))
    return _csr(np.concatenate(rows), np.concatenate(cols), n ** 3)


def hub_pattern(nb, widths):
    """A chain; the hub of each width is coupled, both ways, to that many rows
    before it, so its own search and those around it reach them."""
    i = np.arange(nb)
    rows, cols = [i, i[1:], i[:-1]], [i, i[:-1], i[1:]]
    at = 100
    for w in widths:
        at += w + 50
        far = np.arange(at - w, at - 1)
        rows += [np.full(far.size, at), far]
        cols += [far, np.full(far.size, at)]
    assert at < nb
    return _csr(np.concatenate(rows), np.concatenate(cols), nb)


@pytest.mark.parametrize("k", [0, 1, 2, 3, 4])
def test_grid(api, oracle_mod, k):  # noqa: F811
    Ap, Aj = synth.stencil7_pattern(30, 29, 31)
    check_vs_oracle(api, oracle_mod, "grid", Ap.size - 1, Ap, Aj, k)


def test_grid_27_points(api, oracle_mod):  # noqa: F811
    Ap, Aj = stencil27_pattern(30)
    check_vs_oracle(api, oracle_mod, "27 points", Ap.size - 1, Ap, Aj, 1)


# first tables of 64, 64, 128 and 256 slots, and the largest at once
@pytest.mark.parametrize("k", [0, 1, 4, 5, 7])
def test_hubs(api, oracle_mod, k):  # noqa: F811
    nb = 25000
    Ap, Aj = hub_pattern(nb, [40, 43, 44, 45, 46, 47, 48, 49, 90, 93, 94, 95, 96, 97, 185, 188, 189, 190, 191, 192, 193,
                              300, 600])
    check_vs_oracle(api, oracle_mod, "hubs", nb, Ap, Aj, k)


def _seconds(f):
    f()
    times = []
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    return min(times)


def test_search_cost_of_wide_rows(api):  # noqa: F811
    """27 points, k = 3: the rows reach several hundred vertices.  About twice
    the time of k = 0; a table filled to its last slot first made it 30 times."""
    Ap, Aj = (cuda_i32(a) for a in stencil27_pattern(10))
    assert _seconds(lambda: api.symbolic_device(Ap, Aj, 3)) < 8 * _seconds(lambda: api.symbolic_device(Ap, Aj, 0))


def test_level_cost_of_long_column_lists(api):  # noqa: F811
    """27 points, k = 4: the level sets of L^T, whose lists come in no certain
    order, take about 0.6 of those of L; waiting for them entry by entry in that
    order they took twice as long."""
    Ap, Aj = (cuda_i32(a) for a in stencil27_pattern(10))
    Pp, Pj, _ = api.symbolic_device(Ap, Aj, 4)
    assert _seconds(lambda: api.levels_device(Pp, Pj, 3)) < 1.3 * _seconds(lambda: api.levels_device(Pp, Pj, 0))


@pytest.mark.parametrize("width", [35, 36, 37, 71, 72, 73, 109])
def test_list_edges(api, oracle_mod, width):  # noqa: F811
    """Lists of about as many rows as are listed at a time, and twice and three
    times as many."""
    nb = 2 * width + 5
    Ap, Aj = wide_row_pattern(nb, width)
    for k in (0, 2):
        check_vs_oracle(api, oracle_mod, f"wide{width}", nb, Ap, Aj, k)

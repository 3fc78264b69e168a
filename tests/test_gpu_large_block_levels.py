"""Sweeps of block sizes 9..32 where levels hold many rows: one, four and eight
rows to a ticket, on both sides of the limits between them, groups of rows that
straddle two levels and read each other.  Against the oracle (relative 1e-12) and
the bits of the point-granularity application."""
import numpy as np
import pytest
import torch

from test_gpu_large_blocks import api, cuda, rel  # noqa: F401

pytestmark = pytest.mark.gpu


def layers(m, bs, seed):
    """Three layers of m block rows, every row coupled both ways to two of the
    layer before: the first of a layer to the last of the one before."""
    i = np.arange(3 * m)
    rows, cols = [i], [i]
    for layer in (1, 2):
        j = np.arange(m)
        for back in (j, (7 * j + 3) % m):
            lo, up = layer * m - 1 - back, layer * m + j
            rows += [up, lo]
            cols += [lo, up]
    key = np.unique(np.concatenate(rows) * 3 * m + np.concatenate(cols))
    rows, cols = key // (3 * m), key % (3 * m)
    Ap = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=3 * m))]).astype(np.int32)
    Ax = np.random.default_rng(seed).uniform(-0.1, 0.1, (rows.size, bs, bs))
    Ax[rows == cols] += 4.0 * np.eye(bs)
    return 3 * m, Ap, cols.astype(np.int32), Ax.ravel()


# six levels' rows for 4 and 8 wavefronts of each of 256 compute units: 171 and
# 342 rows a level
@pytest.mark.parametrize("bs", [9, 25, 32])
@pytest.mark.parametrize("m", [41, 170, 171, 341, 342, 683, 1000])
def test_rows_of_a_ticket(api, oracle_mod, m, bs):  # noqa: F811
    nb, Ap, Aj, Ax = layers(m, bs, seed=m + bs)
    O = oracle_mod.OracleILU(nb, bs, Ap, Aj, 0).factor(Ax)
    M = api.BlockILU(nb, bs, Ap, Aj, 0)
    assert M.factor(cuda(Ax)) == -1
    for seed in (1, 2, 3):
        r = np.random.default_rng(seed).standard_normal(nb * bs)
        z = M.apply(cuda(r))
        assert rel(z.cpu().numpy(), O.apply(r)) <= 1e-12
        assert torch.equal(M.apply_point(cuda(r)), z)
    M.check()
    M.close()


def test_wide_levels_cost(api):  # noqa: F811
    """20000 rows a level: the sweeps take about 0.9 of the point rows' time, where
    a ticket for every row made it ten times as much."""
    bs = 9
    nb, Ap, Aj, Ax = layers(20000, bs, seed=1)
    M = api.BlockILU(nb, bs, Ap, Aj, 0)
    assert M.factor(cuda(Ax)) == -1
    r = cuda(np.random.default_rng(1).standard_normal(nb * bs))

    def us(f):
        f()
        times = []
        for _ in range(7):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            f()
            e[1].record()
            torch.cuda.synchronize()
            times.append(1e3 * e[0].elapsed_time(e[1]))
        return min(times)

    z = M.apply(r)
    assert torch.equal(M.apply_point(r), z)
    block, point = us(lambda: M.apply(r, out=z)), us(lambda: M.apply_point(r, out=z))
    print(f"[large block] 60000 rows, b = 9: {block:.0f} us by block rows, {point:.0f} us by point rows", flush=True)
    assert block < 1.2 * point
    M.close()

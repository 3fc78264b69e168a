"""Pencil sweeps (the default sweeps on patterns with grid lines) on the GPU:
the bits of the row-tile sweeps and the oracle's values at the edges of their
tiles, for several columns, both precisions and the transposed pair; column
passes of bilu_apply_noalloc; graph replays; an expired wait is reported and
leaves the next application unharmed."""
import numpy as np
import pytest
import torch

from paper_1703_01325_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1703_01325_amd import api as A
    return A


def _pair(api, s, k, precision="fp64"):
    """The same system with the default sweeps and with row tiles."""
    Ax = torch.from_numpy(s.Ax).cuda()
    out = []
    for group in (None, 1):
        M = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, k, transpose=True)
        M.tune(tile_group=group)
        assert M.factor(Ax, precision=precision) == -1
        out.append(M)
    return out


# lines of two cells, one plane, one line per plane, a tile exactly, one line
# more, several blocks each way with remainders; 3, 6, 11 and 21 dependency
# slots; every block size
CASES = [((2, 2, 2), 3, 0), ((7, 9, 1), 3, 1), ((5, 2, 11), 2, 1), ((6, 7, 3), 3, 0), ((6, 8, 4), 3, 0),
         ((33, 17, 13), 3, 1), ((9, 16, 10), 1, 2), ((12, 11, 10), 1, 3), ((8, 9, 10), 2, 3), ((5, 12, 9), 4, 2),
         ((70, 5, 6), 4, 0), ((6, 7, 8), 5, 1), ((5, 6, 7), 6, 1), ((5, 7, 6), 7, 0), ((4, 5, 7), 8, 1)]


@pytest.mark.parametrize("grid,b,k", CASES, ids=[f"{'x'.join(map(str, g))}_b{b}_k{k}" for g, b, k in CASES])
def test_pencil_bits_of_row_tiles(api, oracle_mod, grid, b, k):
    s = synth.reservoir(*grid, b, seed=31)
    O = oracle_mod.OracleILU(s.nb, s.bs, s.Ap, s.Aj, k).factor(s.Ax)
    rng = np.random.default_rng(b + 10 * k)
    for precision in ("fp64", "fp32"):
        M, P = _pair(api, s, k, precision)
        for R in (1, 2, 3):
            r = torch.from_numpy(rng.standard_normal(s.n if R == 1 else (s.n, R))).cuda()
            for tr in (False, True):
                ref = P.apply(r, transpose=tr)
                for _ in range(2):
                    assert torch.equal(M.apply(r, transpose=tr), ref)
                if precision == "fp64" and not tr:
                    rc, zc = r.cpu().numpy().reshape(s.n, R), ref.cpu().numpy().reshape(s.n, R)
                    for j in range(R):
                        zo = O.apply(np.ascontiguousarray(rc[:, j]))
                        assert np.abs(zc[:, j] - zo).max() <= 1e-12 * np.abs(zo).max()
        M.check()
        M.close()
        P.close()


def test_pencil_column_pairs(api):
    """Enough tiles times columns that two columns are swept together."""
    s = synth.reservoir(4, 60, 60, 3, seed=5)
    for k in (0, 1):
        M, P = _pair(api, s, k)
        for R in (16, 30):
            r = torch.from_numpy(synth.multi_rhs(s.n, R)).cuda()
            for tr in (False, True):
                assert torch.equal(M.apply(r, transpose=tr), P.apply(r, transpose=tr))
        M.check()


def test_pencil_special_values(api):
    """Infinities, NaN and the not-ready pattern in the right-hand side go
    through as through the row tiles."""
    s = synth.reservoir(9, 10, 11, 3, seed=8)
    M, P = _pair(api, s, 1)
    r = torch.randn(s.n, dtype=torch.float64, device="cuda")
    r[5], r[600], r[1800] = float("inf"), float("nan"), -0.0
    r.view(torch.int64)[2500] = 0x7FF4DEADBEEF1234
    a, b = M.apply(r), P.apply(r)
    assert torch.equal(a.view(torch.int64), b.view(torch.int64))
    ok = torch.randn(s.n, dtype=torch.float64, device="cuda")
    assert torch.equal(M.apply(ok), P.apply(ok))
    M.check()


def test_pencil_noalloc_columns(api):
    """Several columns before any bilu_apply of as many: one after the other
    in the room the factorisation made."""
    from paper_1703_01325_amd import _native as N
    s = synth.reservoir(9, 10, 11, 3, seed=9)
    M, P = _pair(api, s, 1)
    r = torch.from_numpy(synth.multi_rhs(s.n, 5)).cuda()
    z = torch.empty_like(r)
    N.bilu_apply_noalloc(M._ctx, r.data_ptr(), z.data_ptr(), 5, torch.cuda.current_stream().cuda_stream)
    ref = P.apply(r)
    assert torch.equal(z, ref)
    assert torch.equal(M.apply(r), ref)
    z.zero_()
    N.bilu_apply_noalloc(M._ctx, r.data_ptr(), z.data_ptr(), 5, torch.cuda.current_stream().cuda_stream)
    assert torch.equal(z, ref)
    M.check()


def test_pencil_graph_replay(api):
    s = synth.reservoir(20, 21, 22, 3, seed=10)
    M, P = _pair(api, s, 0)
    r = torch.randn(s.n, dtype=torch.float64, device="cuda")
    z = torch.empty_like(r)
    M.apply(r, out=z)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        M.apply(r, out=z)
    for i in range(4):
        r.copy_(torch.randn(s.n, dtype=torch.float64, device="cuda"))
        z.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, P.apply(r)), i
        assert torch.equal(M.apply(r), z), i
    M.check()


def test_pencil_expired_wait(api):
    from paper_1703_01325_amd import _native as N
    s = synth.reservoir(12, 20, 20, 3, seed=11)
    M, P = _pair(api, s, 1)
    r = torch.randn(s.n, dtype=torch.float64, device="cuda")
    M.tune(spin_limit=1)
    M.apply(r)
    with pytest.raises(N.BiluError) as ei:
        M.check()
    assert ei.value.code == N.ERR_TIMEOUT
    M.tune(spin_limit=0)
    for _ in range(2):
        assert torch.equal(M.apply(r), P.apply(r))
    M.check()

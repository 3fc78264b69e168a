"""Pencil sweeps that are known to be pencil sweeps against row tiles that are
known to be row tiles, bit for bit: the widest rows of every block size, two
columns together, and batches of every block size in both precisions, with
members factored anew and after the layout was chosen again."""
import numpy as np
import pytest
import torch

from paper_1703_01325_amd import synth

from test_gpu_batch import api, cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def _pair(api, s, k, precision):  # noqa: F811
    """The same factors swept by pencils and by row tiles."""
    Ax = cuda(s.Ax)
    out = []
    for group, form in ((None, "pencils"), (1, "tiles")):
        M = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, k, transpose=True)
        M.tune(tile_group=group)
        assert M.factor(Ax, precision=precision) == -1
        for tr in (False, True):
            assert M.sweep_info(1, transpose=tr)["form"] == (form, form)
        out.append(M)
    return out


# 11 and 21 dependency slots; blocks of lines with remainders both ways
WIDE = [((6, 13, 9), b, 2) for b in range(1, 9)] + [((6, 13, 9), b, 3) for b in range(1, 5)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("grid,b,k", WIDE, ids=[f"b{b}k{k}" for _, b, k in WIDE])
def test_wide_rows(api, grid, b, k, precision):  # noqa: F811
    s = synth.reservoir(*grid, b, seed=60 + b)
    M, P = _pair(api, s, k, precision)
    for R in (1, 2, 5):
        r = cuda(np.random.default_rng(R).standard_normal(s.n if R == 1 else (s.n, R)))
        for tr in (False, True):
            ref = P.apply(r, transpose=tr)
            for _ in range(2):
                assert torch.equal(M.apply(r, transpose=tr), ref)
    M.check()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("b,k", [(1, 0), (2, 1), (3, 0), (4, 1), (5, 1), (6, 0), (7, 1), (8, 1)])
def test_two_columns_together(api, b, k, precision):  # noqa: F811
    s = synth.reservoir(3, 90, 50, b, seed=70 + b)
    M, P = _pair(api, s, k, precision)
    info = M.sweep_info(32)
    assert info["form"] == ("pencils", "pencils") and info["columns"] == (2, 2)
    r = cuda(np.random.default_rng(b).standard_normal((s.n, 32)))
    for tr in (False, True):
        assert torch.equal(M.apply(r, transpose=tr), P.apply(r, transpose=tr))
    M.check()


# ---- batches ---------------------------------------------------------------
GRIDS = [((4, 9, 1), 3), ((6, 8, 4), 2), ((33, 17, 13), 3), ((5, 12, 9), 8), ((2, 21, 20), 1), ((10, 9, 8), 4),
         ((7, 8, 9), 5), ((11, 5, 6), 6), ((5, 6, 7), 7), ((2, 2, 2), 8), ((25, 3, 14), 1), ((3, 30, 2), 5)]


def _batches(api, precision):  # noqa: F811
    """(pencils, tiles, values): the tiles' batch has one member more, without
    grid lines."""
    members = [synth.reservoir(*g, b, seed=90 + i) for i, (g, b) in enumerate(GRIDS)]
    systems = [(m.nb, m.bs, m.Ap, m.Aj) for m in members]
    Ap, Aj = synth.random_block_pattern(40, 0.1, 5)
    extra = np.random.default_rng(6).uniform(-0.1, 0.1, (Aj.size, 4))
    extra[Aj == np.repeat(np.arange(40), np.diff(Ap))] += 5.0 * np.eye(2).ravel()
    Ax = [cuda(m.Ax) for m in members]
    P = api.BlockILUBatch(systems, 0)
    T = api.BlockILUBatch(systems + [(40, 2, Ap, Aj)], 0)
    assert P.factor(Ax, precision=precision) is None
    assert T.factor(Ax + [cuda(extra.ravel())], precision=precision) is None
    assert P.sweep_form() == "pencils" and T.sweep_form() == "tiles"
    return P, T, Ax, cuda(extra.ravel())


def _long(P, T, v):
    return torch.cat([v, torch.ones(T.n - P.n, dtype=torch.float64, device="cuda")])


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_batch(api, precision):  # noqa: F811
    P, T, Ax, extra = _batches(api, precision)
    rng = np.random.default_rng(3)
    for _ in range(3):
        r = cuda(rng.standard_normal(P.n))
        assert torch.equal(P.apply(r), T.apply(_long(P, T, r))[:P.n])
    b = cuda(rng.standard_normal(P.n))
    x, st, info = P.solve(b)
    xt, stt, infot = T.solve(_long(P, T, b))
    assert st == stt and list(info) == list(infot)[:P.nsys] and torch.equal(x, xt[:P.n])
    assert len({i[1] for i in info}) > 1, "members that stop at different steps"


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_batch_member_and_layout(api, precision):  # noqa: F811
    P, T, Ax, extra = _batches(api, precision)
    r = cuda(np.random.default_rng(4).standard_normal(P.n))
    for s in (0, 3, 11):                        # members factored anew by themselves
        for B in (P, T):
            assert B.member(s).factor(2.0 * Ax[s], precision=precision) == -1
    z = P.apply(r)
    assert torch.equal(z, T.apply(_long(P, T, r))[:P.n])
    o = P.offsets
    for s in (2, 3):                            # and applied
        assert torch.equal(P.member(s).apply(r[o[s]:o[s + 1]].contiguous()), z[o[s]:o[s + 1]])
    assert torch.equal(P.apply(r), z)
    tune = P.autotune()                         # through every scale of row tiles and back
    assert tune["candidates"] == 4 and tune["pair_us"] <= tune["default_us"]
    assert P.sweep_form() == ("pencils" if tune["tile_scale"] == 1.0 else "tiles")
    for _ in range(2):
        assert torch.equal(P.apply(r), z)
    assert P.factor(Ax, precision=precision) is None and T.factor(Ax + [extra], precision=precision) is None
    assert torch.equal(P.apply(r), T.apply(_long(P, T, r))[:P.n])


def test_batch_work_space(api):  # noqa: F811
    """A member's own work space (its vector between the sweeps, two exchange
    arrays) is there once the member is applied by itself, not before."""
    members = [synth.reservoir(40, 41, 42, 8, seed=3), synth.reservoir(5, 6, 7, 2, seed=4)]
    P = api.BlockILUBatch([(m.nb, m.bs, m.Ap, m.Aj) for m in members], 0)
    assert P.factor([cuda(m.Ax) for m in members]) is None and P.sweep_form() == "pencils"
    r = cuda(np.random.default_rng(5).standard_normal(P.n))
    z = P.apply(r)
    r0, z0 = r[:members[0].n].clone(), z[:members[0].n].clone()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    m = P.member(0)
    out = m.apply(r0, out=torch.empty_like(z0))
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] >= 8 * members[0].n
    assert torch.equal(out, z0) and torch.equal(P.apply(r), z)

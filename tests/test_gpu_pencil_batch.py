"""Batches swept by pencils (every member a grid, ILU(0)) against the same
members swept by row tiles (a batch with one more member, whose pattern has no
grid lines): the same bits of applications and solves for every block size and
both precisions, with members that stop at different steps, after a member was
factored anew by itself, and after the layout was chosen again."""
import numpy as np
import pytest
import torch

from paper_1703_01325_amd import synth

from test_gpu_batch import api, cuda, small_members  # noqa: F401

pytestmark = pytest.mark.gpu


def _members():
    # a line, a plane, one tile exactly, several blocks of lines with remainders
    out = small_members()
    out += [synth.reservoir(*g, b, seed=90 + b) for g, b in (((9, 1, 1), 2), ((4, 9, 1), 3), ((6, 8, 4), 2),
                                                             ((33, 17, 13), 3), ((5, 12, 9), 8), ((2, 21, 20), 1))]
    return out


def _random_member(nb=40, b=2):
    Ap, Aj = synth.random_block_pattern(nb, 0.1, 5)
    Ax = np.random.default_rng(6).uniform(-0.1, 0.1, (Aj.size, b * b))
    Ax[Aj == np.repeat(np.arange(nb), np.diff(Ap))] += 5.0 * np.eye(b).ravel()
    return nb, b, Ap, Aj, Ax.ravel()


def _pair(api, members, precision):  # noqa: F811
    systems = [(m.nb, m.bs, m.Ap, m.Aj) for m in members]
    Ax = [cuda(m.Ax) for m in members]
    nb, b, Ap, Aj, extra = _random_member()
    P = api.BlockILUBatch(systems, 0)
    T = api.BlockILUBatch(systems + [(nb, b, Ap, Aj)], 0)
    assert P.factor(Ax, precision=precision) is None
    assert T.factor(Ax + [cuda(extra)], precision=precision) is None
    return P, T, Ax


def _long(P, T, v):
    """A vector of P's members and ones for T's last member."""
    return torch.cat([v, torch.ones(T.n - P.n, dtype=torch.float64, device="cuda")])


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_pencil_batch_bits_of_row_tiles(api, precision):  # noqa: F811
    members = _members()
    P, T, Ax = _pair(api, members, precision)
    rng = np.random.default_rng(3)
    for _ in range(3):
        r = cuda(rng.standard_normal(P.n))
        assert torch.equal(P.apply(r), T.apply(_long(P, T, r))[:P.n])
    b = cuda(rng.standard_normal(P.n))
    x, st, info = P.solve(b)
    xt, stt, infot = T.solve(_long(P, T, b))
    assert st == stt and list(info) == list(infot)[:P.nsys] and torch.equal(x, xt[:P.n])
    assert len({i[1] for i in info}) > 1, "members that stop at different steps"


def test_pencil_batch_member_and_layout(api):  # noqa: F811
    members = _members()
    P, T, Ax = _pair(api, members, "fp64")
    r = cuda(np.random.default_rng(4).standard_normal(P.n))
    rt = _long(P, T, r)
    for s in (0, 13):
        for B in (P, T):
            assert B.member(s).factor(2.0 * Ax[s]) == -1
    z = P.apply(r)
    assert torch.equal(z, T.apply(rt)[:P.n])
    o = P.offsets
    assert torch.equal(P.member(13).apply(r[o[13]:o[14]].contiguous()), z[o[13]:o[14]])
    tune = P.autotune()
    assert tune["candidates"] == 4 and tune["pair_us"] <= tune["default_us"]
    for _ in range(2):
        assert torch.equal(P.apply(r), z)
    assert P.factor(Ax) is None and T.factor(Ax + [cuda(_random_member()[4])]) is None
    assert torch.equal(P.apply(r), T.apply(rt)[:P.n])

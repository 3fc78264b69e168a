"""Block sizes 9..32 at the edges of their kernels -- 1 to 4 elements of a
block per thread (16 | 17, 22 | 23, 27 | 28, 32), one to three update pairs at
once (9, 11 | 12) -- against the oracle: factors and applications relative
1e-12, a zero pivot reported at its row."""
import numpy as np
import pytest
import torch

from paper_1703_01325_amd import synth

from test_gpu_large_blocks import api, cuda, rel  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bs,k", [(9, 2), (11, 1), (12, 1), (16, 2), (17, 1), (22, 0), (23, 1), (27, 0), (28, 1),
                                  (32, 0), (32, 1)])
def test_large_block_edges(api, oracle_mod, bs, k):  # noqa: F811
    for grid in ((4, 3, 3), (1, 1, 1), (7, 1, 2)):
        s = synth.reservoir(*grid, bs, seed=300 + bs)
        O = oracle_mod.OracleILU(s.nb, s.bs, s.Ap, s.Aj, k).factor(s.Ax)
        M = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, k)
        for _ in range(2):
            assert M.factor(cuda(s.Ax)) == -1
            F, D = M.factors()
            assert rel(F.cpu().numpy(), O.F) <= 1e-12 and rel(D.cpu().numpy(), O.Dinv) <= 1e-12
            for seed in (1, 2):
                r = np.random.default_rng(seed).standard_normal(s.n)
                z = M.apply(cuda(r))
                assert rel(z.cpu().numpy(), O.apply(r)) <= 1e-12
                assert torch.equal(M.apply_point(cuda(r)), z)
        M.check()


@pytest.mark.parametrize("bs", [9, 17, 32])
def test_large_block_permuted_and_zero_pivots(api, oracle_mod, bs):  # noqa: F811
    s = synth.reservoir(3, 3, 2, bs, seed=350 + bs)
    Ax = s.Ax.reshape(-1, bs, bs).copy()
    diag = np.flatnonzero(s.Aj == np.repeat(np.arange(s.nb), np.diff(s.Ap)))
    Ax[diag] = Ax[diag][:, :, ::-1]                  # rows of the diagonal blocks reversed: every step swaps
    M = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, 0)
    assert M.factor(cuda(Ax.ravel())) == -1
    O = oracle_mod.OracleILU(s.nb, s.bs, s.Ap, s.Aj, 0).factor(Ax.ravel())
    assert rel(M.factors()[1].cpu().numpy(), O.Dinv) <= 1e-12
    Ax[diag[4]] = 0.0
    Ax[s.Ap[4]:s.Ap[5]] = 0.0
    assert M.factor(cuda(Ax.ravel())) == 4

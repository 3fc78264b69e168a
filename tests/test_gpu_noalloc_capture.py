"""bilu_apply_noalloc on a grid pattern works in nothing of the context's that
another call may move or share: a captured call gives the bits of bilu_apply
after applications and solves of more columns, and a call may run beside
bilu_apply of the same context on another stream."""
import pytest
import torch

from paper_1703_01325_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1703_01325_amd import api as A
    return A


def _noalloc(M, r, z):
    from paper_1703_01325_amd import _native as N
    N.bilu_apply_noalloc(M._ctx, r.data_ptr(), z.data_ptr(), 1 if r.dim() == 1 else r.shape[1],
                         torch.cuda.current_stream().cuda_stream)


@pytest.mark.parametrize("R", [1, 3])
def test_captured_noalloc_after_wider_calls(api, R):
    s = synth.reservoir(13, 12, 11, 3, seed=21)
    Ax = torch.from_numpy(s.Ax).cuda()
    M = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, 1)
    assert M.factor(Ax) == -1
    gen = torch.Generator(device="cuda").manual_seed(R)

    def draw(cols):
        return torch.randn((s.n,) if cols == 1 else (s.n, cols), generator=gen, dtype=torch.float64, device="cuda")

    r, z = draw(R), torch.empty((s.n,) if R == 1 else (s.n, R), dtype=torch.float64, device="cuda")
    _noalloc(M, r, z)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _noalloc(M, r, z)
    for cols in (None, 8, 16, 32, 1):
        if cols:
            wide = draw(cols)
            M.apply(wide)
            M.solve(Ax, wide, maxit=2)
            assert M.factor(Ax) == -1
        r.copy_(draw(R))
        z.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, M.apply(r)), cols
    M.check()
    M.close()


def test_noalloc_beside_apply(api):
    s = synth.reservoir(24, 25, 26, 3, seed=22)
    Ax = torch.from_numpy(s.Ax).cuda()
    M = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, 0)
    assert M.factor(Ax) == -1
    r1, r2 = (torch.randn(s.n, dtype=torch.float64, device="cuda") for _ in range(2))
    want1, want2 = M.apply(r1), M.apply(r2)
    z1, z2 = torch.empty_like(r1), torch.empty_like(r2)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(10):
        with torch.cuda.stream(side):
            for _ in range(4):
                _noalloc(M, r1, z1)
        for _ in range(4):
            M.apply(r2, out=z2)
        torch.cuda.synchronize()
        assert torch.equal(z1, want1) and torch.equal(z2, want2)
    M.check()
    M.close()

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


LAUNCH_KNOBS = [dict(helper=True), dict(helper=False), dict(rhs_pairs=True), dict(split_dinv=True),
                dict(split_dinv=False), dict(fuse_spmv=True), dict(blocks=7)]
DEFAULTS = dict(helper="auto", rhs_pairs="auto", split_dinv="auto", fuse_spmv=False, blocks=0)


@pytest.mark.parametrize("knob", LAUNCH_KNOBS, ids=[f"{k}-{v}" for d in LAUNCH_KNOBS for k, v in d.items()])
def test_noalloc_after_a_launch_knob(api, knob):
    """A knob that shapes no layout, set or cleared after the factorisation,
    does not take the layouts away."""
    s = synth.reservoir(9, 10, 11, 3, seed=23)
    Ax = torch.from_numpy(s.Ax).cuda()
    r = torch.randn(s.n, dtype=torch.float64, device="cuda")
    P = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, 1)
    assert P.factor(Ax) == -1
    want = P.apply(r)
    for before, after in (({}, knob), (knob, {k: DEFAULTS[k] for k in knob})):
        M = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, 1)
        M.tune(**before)
        assert M.factor(Ax) == -1
        M.tune(**after)
        z = torch.empty_like(r)
        _noalloc(M, r, z)
        assert torch.equal(z, want)
        M.check()
        M.close()


def test_noalloc_after_another_layout_is_asked_for(api):
    """A knob that asks for other layouts leaves none that hold the factors
    (until an application lays them out)."""
    from paper_1703_01325_amd import _native as N
    s = synth.reservoir(9, 10, 11, 3, seed=24)
    r = torch.randn(s.n, dtype=torch.float64, device="cuda")
    z = torch.empty_like(r)
    for knob in (dict(tile_rows=17), dict(tile_block=(2, 3)), dict(mode=1)):
        M = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, 1)
        assert M.factor(torch.from_numpy(s.Ax).cuda()) == -1
        M.tune(**knob)
        with pytest.raises(N.BiluError) as ei:
            _noalloc(M, r, z)
        assert ei.value.code == N.ERR_STATE
        want = M.apply(r)
        _noalloc(M, r, z)
        assert torch.equal(z, want)
        M.check()
        M.close()


@pytest.mark.parametrize("call", ["noalloc", "apply", "transpose"])
@pytest.mark.parametrize("before,after", [({}, dict(helper=True)), (dict(split_dinv=False), dict(split_dinv="auto"))],
                         ids=["pencils", "tiles"])
def test_replay_after_a_launch_knob_and_a_factorisation(api, call, before, after):
    """A captured application reads the factors of the last factorisation, also
    where a launch knob has made later ones take the other form."""
    s = synth.reservoir(11, 9, 10, 3, seed=25)
    Ax = torch.from_numpy(s.Ax).cuda()
    M = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, 0, transpose=True)
    P = api.BlockILU(s.nb, s.bs, s.Ap, s.Aj, 0, transpose=True)
    M.tune(**before)
    assert M.factor(Ax) == -1
    r = torch.randn(s.n, dtype=torch.float64, device="cuda")
    z = torch.empty_like(r)

    def run(B, out):
        if call == "noalloc":
            _noalloc(B, r, out)
        else:
            B.apply(r, out=out, transpose=call == "transpose")

    run(M, z)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run(M, z)
    M.tune(**after)
    for scale in (2.0, 0.5, 3.0):
        values = scale * Ax
        assert M.factor(values) == -1 and P.factor(values) == -1
        want = torch.empty_like(r)
        run(P, want)
        for _ in range(2):
            z.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(z, want)
            assert torch.equal(M.apply(r, transpose=call == "transpose"), want)
    M.check()


@pytest.mark.parametrize("grid,b,k,R", [((60, 220, 85), 3, 0, 1), ((31, 33, 42), 3, 1, 32), ((19, 21, 40), 8, 0, 32),
                                        ((70, 70, 70), 1, 0, 12)],
                         ids=["1col", "32cols", "b8", "b1"])
def test_noalloc_near_the_scratch_limit(api, grid, b, k, R):
    """Vectors and exchange arrays of close to the most columns the call takes."""
    Ap, Aj = synth.stencil7_pattern(*grid)
    nb = Ap.size - 1
    assert 0.75 * 2 ** 25 < 8 * nb * b * R <= 2 ** 25 - 256
    gen = torch.Generator(device="cuda").manual_seed(R)
    rows = torch.repeat_interleave(torch.arange(nb), torch.from_numpy(Ap).diff())
    Ax = 0.1 * torch.randn(Aj.size, b, b, generator=gen, dtype=torch.float64, device="cuda")
    Ax[(torch.from_numpy(Aj) == rows).cuda()] += (2.0 + b) * torch.eye(b, dtype=torch.float64, device="cuda")
    M = api.BlockILU(nb, b, Ap, Aj, k)
    assert M.factor(Ax.reshape(-1)) == -1
    assert M.sweep_info(R)["form"] == ("pencils", "pencils")
    r = torch.randn((nb * b,) if R == 1 else (nb * b, R), generator=gen, dtype=torch.float64, device="cuda")
    z = torch.empty_like(r)
    for _ in range(2):
        z.zero_()
        _noalloc(M, r, z)
        assert torch.equal(z, M.apply(r))
    M.check()
    M.close()

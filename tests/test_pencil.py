"""Pencil layouts on the host."""
import pytest

from paper_1703_01325_amd import synth


@pytest.fixture(scope="module")
def N():
    from paper_1703_01325_amd import _native
    return _native


@pytest.mark.parametrize("grid", [(2, 2, 2), (7, 9, 1), (5, 2, 11), (6, 7, 3), (6, 8, 4), (33, 17, 13), (5, 40, 30)])
def test_pencil_layouts_validate(N, grid):
    """The host self-check builds and walks the pencil layouts of every sweep
    (every row once, every LDS place decoded to the row it holds when read)."""
    Ap, Aj = synth.stencil7_pattern(*grid)
    for bs in range(1, 9):
        for k in (0, 1, 2, 3):
            ctx = N.bilu_analyze(Ap.size - 1, bs, Ap, Aj, k, N.WANT_TRANSPOSE)
            N.bilu_validate(ctx)
            N.bilu_destroy(ctx)

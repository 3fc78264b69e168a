"""The form of an application's sweeps as reported, on the host: pencils on every
grid in natural order up to the widest rows of their kernels, row tiles where a
pattern has no grid lines or a knob asks for them."""
import numpy as np
import pytest

from paper_1703_01325_amd import synth

GRIDS = [(2, 2, 2), (7, 9, 1), (5, 2, 11), (6, 7, 3), (6, 8, 4), (33, 17, 13), (5, 40, 30)]


@pytest.fixture(scope="module")
def api():
    from paper_1703_01325_amd import api as A
    return A


@pytest.mark.parametrize("grid", GRIDS, ids=["x".join(map(str, g)) for g in GRIDS])
def test_grids_are_swept_by_pencils(api, grid):
    Ap, Aj = synth.stencil7_pattern(*grid)
    for bs in range(1, 9):
        for k in (0, 1, 2, 3):
            M = api.BlockILU(Ap.size - 1, bs, Ap, Aj, k, transpose=True)
            widest = 0
            Pp, Pj, _ = M.pattern()
            rows = np.repeat(np.arange(Ap.size - 1), np.diff(Pp))
            for side in (Pj < rows, Pj > rows):
                widest = max(widest, int(np.bincount(rows[side], minlength=1).max()))
            # (lines of two cells: the fill of k = 2 couples the end of a line
            # with the start of the next, rows one apart, so there are no lines)
            fits = (widest <= 11 or (widest <= 21 and bs <= 4)) and not (grid[0] == 2 and k >= 2)
            for tr in (False, True):
                for nrhs in (1, 2, 32):
                    info = M.sweep_info(nrhs, transpose=tr)
                    if not fits:
                        assert info["form"] == ("tiles", "tiles")
                        continue
                    assert info["form"] == ("pencils", "pencils"), (bs, k, tr, nrhs)
                    assert all(widest <= w <= 21 and t >= 1 for w, t in zip(info["width"], info["tiles"]))
            M.close()


def test_other_patterns_are_swept_by_row_tiles(api):
    line = synth.stencil7_pattern(9, 1, 1)
    cell = synth.stencil7_pattern(1, 1, 1)
    for Ap, Aj in (line, cell, synth.random_block_pattern(60, 0.1, 5)):
        M = api.BlockILU(Ap.size - 1, 2, Ap, Aj, 0)
        assert M.sweep_info()["form"] == ("tiles", "tiles")


def test_knobs_and_refusals(api):
    from paper_1703_01325_amd import _native as N
    Ap, Aj = synth.stencil7_pattern(6, 7, 5)
    M = api.BlockILU(Ap.size - 1, 3, Ap, Aj, 0)
    for on, off in ((dict(tile_rows=16), dict(tile_rows=0)), (dict(tile_group=1), dict(tile_group=0)),
                    (dict(helper=True), dict(helper="auto")), (dict(split_dinv=True), dict(split_dinv="auto")),
                    (dict(fuse_spmv=True), dict(fuse_spmv=False)), (dict(blocks=8), dict(blocks=0))):
        M.tune(**on)
        assert M.sweep_info()["form"] == ("tiles", "tiles")
        M.tune(**off)
        assert M.sweep_info()["form"] == ("pencils", "pencils")
    M.tune(mode=1)
    assert M.sweep_info()["form"] == ("levels", "levels")
    M.tune(mode=2, line_sweep=(7, 3))
    assert M.sweep_info()["form"] == ("lines", "lines")
    for args, code in (((0, False), N.ERR_ARG), ((33, False), N.ERR_ARG), ((1, True), N.ERR_STATE)):
        with pytest.raises(N.BiluError) as ei:
            M.sweep_info(*args)
        assert ei.value.code == code
    L = api.BlockILU(Ap.size - 1, 9, Ap, Aj, 0)
    assert L.sweep_info()["form"] == ("rows", "rows")
    with pytest.raises(N.BiluError):
        L.sweep_info(2)


def test_batch_form(api):
    grids = [synth.reservoir(*g, b, seed=1) for g, b in (((4, 5, 6), 3), ((7, 3, 2), 8))]
    systems = [(m.nb, m.bs, m.Ap, m.Aj) for m in grids]
    Ap, Aj = synth.random_block_pattern(40, 0.1, 5)
    assert api.BlockILUBatch(systems, 0).sweep_form() == "pencils"
    assert api.BlockILUBatch(systems + [(40, 2, Ap, Aj)], 0).sweep_form() == "tiles"
    assert api.BlockILUBatch(systems, 1).sweep_form() == "tiles"

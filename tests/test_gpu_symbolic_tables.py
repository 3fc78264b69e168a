"""GPU symbolic phase at the edges of its tables and lists: rows whose search
just fits, or outgrows, the first tables (48 and 96 vertices), the second
(192) and the largest (768, refused beyond), and level sets of rows that read
more rows than a lane polls at once (12) or lists before its first wait (32).
Integer work: equal to the oracle."""
import numpy as np
import pytest
import torch

from paper_1703_01325_amd import synth

from test_gpu_symbolic import api, check_vs_oracle, cuda_i32  # noqa: F401

pytestmark = pytest.mark.gpu


def wide_row_pattern(nb, width):
    """Tridiagonal, the last row, the last column and row and column nb // 2
    `width` entries wide: the search of the last row reaches about that many
    vertices, a search that passes the middle row as many again."""
    A = np.eye(nb, dtype=bool) | np.eye(nb, k=1, dtype=bool) | np.eye(nb, k=-1, dtype=bool)
    A[nb - 1, nb - width:] = A[nb - width:, nb - 1] = True
    A[nb // 2, :width] = A[:width, nb // 2] = True
    Ap = np.concatenate([[0], np.cumsum(A.sum(1))]).astype(np.int32)
    return Ap, np.nonzero(A)[1].astype(np.int32)


@pytest.mark.parametrize("k", [0, 1, 2, 3])
@pytest.mark.parametrize("width", [12, 13, 32, 33, 47, 48, 49, 96, 97, 191, 192, 193, 600])
def test_table_edges(api, oracle_mod, width, k):  # noqa: F811
    nb = max(2 * width, 70) + 5
    Ap, Aj = wide_row_pattern(nb, width)
    if k and width >= 193:
        nb = width + 7
        Ap, Aj = wide_row_pattern(nb, width // 2)
    check_vs_oracle(api, oracle_mod, f"wide{width}", nb, Ap, Aj, k)


@pytest.mark.parametrize("width,fits", [(765, True), (766, False), (768, False), (769, False)])
def test_largest_table(api, oracle_mod, width, fits):  # noqa: F811
    from paper_1703_01325_amd import _native as N
    Ap, Aj = wide_row_pattern(2000, width)     # the middle row has width + 3 entries
    if fits:
        check_vs_oracle(api, oracle_mod, f"wide{width}", 2000, Ap, Aj, 0)
    else:
        with pytest.raises(N.BiluError):
            api.symbolic_device(cuda_i32(Ap), cuda_i32(Aj), 0)

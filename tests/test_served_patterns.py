"""What the server's sweeps take for granted of the patterns that it generates, and admission checks: at most
two blocks of a row on either side of the diagonal, structural symmetry, and update sets on the diagonal
blocks alone (as many pairs as strictly lower blocks), on the host twin of the generator."""
import numpy as np
import pytest

import oracle


@pytest.mark.parametrize("kind", ["tri", "aniso"])
@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 2), (2, 1), (2, 2), (3, 2), (2, 3), (1, 9), (9, 1), (7, 5), (31, 17)])
def test_generated_patterns(kind, nx, ny):
    from paper_1912_00539_amd import workloads as W
    for seed in (1, 2, 3):
        c = W.request_case(dict(kind=kind, nx=nx, ny=ny, cfl=100.0, seed=seed))
        rows = np.repeat(np.arange(c.n), np.diff(c.rowptr))
        lower, upper = c.colidx < rows, c.colidx > rows
        for side in (lower, upper):
            assert np.bincount(rows[side], minlength=c.n).max(initial=0) <= 2
        pos = set(zip(rows.tolist(), c.colidx.tolist()))
        assert all((j, i) in pos for i, j in pos)
        assert oracle.pairs(c.n, c.rowptr, c.colidx)[0][-1] == lower.sum()

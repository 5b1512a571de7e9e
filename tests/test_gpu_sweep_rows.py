"""Synchronous factor sweeps on patterns with diagonal update sets, rows of more than three blocks a side and
far neighbours, on either side of the sizes where a quad per row takes the sweep instead of a quad per
block: the rows of a mesh appended to with three mutually neighbouring cells, whose update sets off the
diagonal keep the quad per block, come out the same, bit for bit, with the same flags."""
import numpy as np
import pytest

from tests.test_gpu_factor_forms import with_clique

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,nx,ny", [("f64", 440, 450), ("f64", 460, 450), ("f32", 840, 850), ("f32", 860, 850)])
def test_rows_equal_blocks(prec, nx, ny):
    import torch
    from paper_1912_00539_amd import workloads as W
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = W.case("quad", seed=3, nx=nx, ny=ny, order="random")
    rows = np.repeat(np.arange(c.n), np.diff(c.rowptr))
    diag = np.flatnonzero(rows == c.colidx)
    assert np.diff(c.rowptr).max() == 5 and max(np.bincount(rows[c.colidx < rows])) > 3
    c.vals[diag[[7, c.n // 2]]] = 0.0
    a, b = DeviceSystem(c, prec=prec, restart=0), DeviceSystem(with_clique(c), prec=prec, restart=0)
    for nsw, init in ((1, "A"), (2, "A"), (1, "LU"), (2, "LU")):
        out = []
        for s in (a, b):
            s.work.fill_(0)
            s.factor(nsw, "sync", init=init)
            csr = torch.empty_like(s.LU)
            from paper_1912_00539_amd import abilu as L
            L.abilu_factor_to_csr(s.pattern, prec, s.LU, csr)
            out.append((csr[: 16 * c.nnzb].nan_to_num(), s.Dinv[: 16 * c.n].nan_to_num(), s.flags(clear=True)))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]), (nsw, init)
        assert out[0][2] == out[1][2], (nsw, init)

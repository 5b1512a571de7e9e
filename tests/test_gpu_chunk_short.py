"""Chunked sweeps on short chains, where the number of rows and of chunks decides between forms: in the
application sixteen lanes or a quad per chunk, in the factor two launches or whole rows, sweep by sweep.
Against the workgroup-per-chunk runner, bit for bit, on either side of each line."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def lines(kind):
    from paper_1912_00539_amd import workloads as W
    if kind == "aniso":
        return W.case("aniso", seed=2, nx=149, ny=151, order="line")
    nx, ny, nz = 20, 20, 61
    q = np.arange(nx * ny * nz).reshape(nx, ny, nz)
    fa = np.concatenate([q[:-1].ravel(), q[:, :-1].ravel(), q[:, :, :-1].ravel()])
    fb = np.concatenate([q[1:].ravel(), q[:, 1:].ravel(), q[:, :, 1:].ravel()])
    m = W.Mesh(q.size, fa, fb, np.ones(fa.size), "lines3", (nx, ny, nz))
    return W.assemble(m, W.natural_order(m), 3, "cfl", cfl=50.0)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind", ["aniso", "lines3"])
def test_short_chains(kind, prec):
    import torch
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = lines(kind)
    a, b = DeviceSystem(c, prec=prec), DeviceSystem(c, prec=prec)
    for s in (a, b):
        s.factor(2, "sync")
    for R in (1, 2, 3, 4, 5, 6, 7, 9, 10, 16):
        assert a.set_chunks(R, "rows")["runner"] == "rows" and b.set_chunks(R, "levels")["runner"] == "levels"
        for nsw in (1, 3):
            z = [torch.full_like(s.b, float("nan")) for s in (a, b)]
            for s, v in zip((a, b), z):
                s.work.fill_(255)
                s.apply(s.b, v, nsw, "chunk_sync")
            assert torch.equal(*z), (R, nsw)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind", ["aniso", "lines3"])
def test_short_chains_factor(kind, prec):
    import torch
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = lines(kind)
    rows = np.repeat(np.arange(c.n), np.diff(c.rowptr))
    c.vals = c.vals.copy()
    c.vals[np.flatnonzero(rows == c.colidx)[[5, c.n // 2]]] = 0.0   # singular blocks raise their flag once
    a, b = DeviceSystem(c, prec=prec), DeviceSystem(c, prec=prec)
    for R in (1, 2, 3, 4, 8, 24):
        assert a.set_chunks(R, "rows")["runner"] == "rows" and b.set_chunks(R, "levels")["runner"] == "levels"
        for nsw, init in ((1, "A"), (2, "A"), (3, "A"), (1, "LU"), (2, "LU")):
            for s in (a, b):
                if init == "A":
                    s.LU.fill_(float("nan"))
                    s.Dinv.fill_(float("nan"))
                s.work.fill_(0)
                s.factor(nsw, "chunk_sync", init=init)
            assert torch.equal(a.LU.nan_to_num(), b.LU.nan_to_num()), (R, nsw, init)
            assert torch.equal(a.Dinv.nan_to_num(), b.Dinv.nan_to_num()), (R, nsw, init)
            assert a.flags(clear=True) == b.flags(clear=True), (R, nsw, init)

"""Chunked sweeps on chunks that are chains (rows whose only neighbours inside their chunk are the rows
next to them): the sixteen-lane form against the workgroup-per-chunk runner, bit for bit, at chunk
lengths around its steps of four and sixteen rows, with one to three blocks a side."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def lines(kind):
    from paper_1912_00539_amd import workloads as W
    if kind == "chain":       # a row before, a row after
        return W.case("chain", seed=1, n=101)
    if kind == "grid":        # and one line on each side
        return W.case("aniso", seed=2, nx=7, ny=45, order="line")
    nx, ny, nz = 4, 3, 37     # lines of nz cells, neighbours in two directions
    q = np.arange(nx * ny * nz).reshape(nx, ny, nz)
    fa = np.concatenate([q[:-1].ravel(), q[:, :-1].ravel(), q[:, :, :-1].ravel()])
    fb = np.concatenate([q[1:].ravel(), q[:, 1:].ravel(), q[:, :, 1:].ravel()])
    m = W.Mesh(q.size, fa, fb, np.ones(fa.size), "lines3", (nx, ny, nz))
    return W.assemble(m, W.natural_order(m), 3, "cfl", cfl=50.0)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind", ["chain", "grid", "lines3"])
@pytest.mark.parametrize("R", [1, 3, 4, 5, 15, 16, 17, 33])
def test_chains_equal_levels(kind, R, prec):
    import torch
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = lines(kind)
    a, b = DeviceSystem(c, prec=prec), DeviceSystem(c, prec=prec)
    assert a.set_chunks(R, "rows")["runner"] == "rows" and b.set_chunks(R, "levels")["runner"] == "levels"

    def same(what):
        assert torch.equal(a.LU, b.LU) and torch.equal(a.Dinv, b.Dinv), what
        assert a.flags(clear=True) == b.flags(clear=True), what
    for s in (a, b):
        s.flags(clear=True)
    for nsw in (1, 2, 3):
        for s in (a, b):
            s.factor(nsw, "chunk_sync")
        same(("from A", nsw))
    for s in (a, b):
        s.A.mul_(1.5)
        s.factor(1, "chunk_sync", init="LU")
    same("from LU")
    for nsw in (1, 2, 3):
        z = [torch.full_like(s.b, float("nan")) for s in (a, b)]
        for s, v in zip((a, b), z):
            s.work.fill_(255)
            s.apply(s.b, v, nsw, "chunk_sync")
        assert torch.equal(*z), nsw

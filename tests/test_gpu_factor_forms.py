"""The row-at-once form of the factor sweeps (patterns whose update sets are the diagonal ones, at most
three lower and three upper blocks a row) against the general form, bit for bit.

Three mutually neighbouring cells appended to a mesh, not connected to it, give its pattern update
sets off the diagonal, so the same system then takes the general form; its rows of the mesh have to
come out the same, in both precisions, for every sweep count, mode and initial guess whose result
does not depend on scheduling, with the same flags where diagonal blocks are singular or need
pivoting."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MESHES = [("chain", dict(n=1)), ("chain", dict(n=2)), ("chain", dict(n=67)), ("tri", dict(nx=1, ny=1)),
          ("tri", dict(nx=9, ny=7)), ("tri", dict(nx=17, ny=15, order="rcm")),
          ("tri", dict(nx=16, ny=9, order="random")), ("quad", dict(nx=13, ny=5)), ("aniso", dict(nx=9, ny=21, order="line")),
          ("random", dict(n=40, deg=0.0))]


def mesh_case(kind, kw):
    from paper_1912_00539_amd import workloads as W
    c = W.case(kind, seed=11, **kw)
    rng = np.random.default_rng(5)
    rows = np.repeat(np.arange(c.n), np.diff(c.rowptr))
    diag = np.flatnonzero(rows == c.colidx)
    c.vals = c.vals.copy()
    for i in rng.permutation(c.n)[:3 + c.n // 20]:   # blocks that need row exchanges
        c.vals[diag[i]] = c.vals[diag[i]][rng.permutation(4)]
    if c.n > 20:                                     # a singular one, and a huge one
        c.vals[diag[7]] = 0.0
        c.vals[diag[13]] *= 1e25
    return c


def with_clique(c):
    from paper_1912_00539_amd.workloads import BSRCase
    n = c.n
    rp = np.concatenate([c.rowptr, c.rowptr[-1] + np.array([3, 6, 9], np.int32)])
    ci = np.concatenate([c.colidx, np.tile(np.arange(n, n + 3, dtype=np.int32), 3)])
    extra = np.tile(np.eye(4), (9, 1, 1)) * np.where(np.arange(9) % 4 == 0, 8.0, 1.0)[:, None, None]
    return BSRCase(n + 3, rp.astype(np.int32), ci.astype(np.int32), np.concatenate([c.vals, extra]),
                   np.concatenate([c.b, np.ones(12)]), dict(c.meta))


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind,kw", MESHES)
def test_row_form_equals_general_form(kind, kw, prec):
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = mesh_case(kind, kw)
    a, b = DeviceSystem(c, prec=prec), DeviceSystem(with_clique(c), prec=prec)
    z = c.nnzb

    def same(what):
        Xa, Da = a.factor_host()
        Xb, Db = b.factor_host()
        assert np.array_equal(Xa, Xb[:z], equal_nan=True) and np.array_equal(Da, Db[:c.n], equal_nan=True), what
        assert a.flags(clear=True) == b.flags(clear=True), what
    for s in (a, b):
        s.flags(clear=True)
    for nsw in (1, 2, 3):
        for s in (a, b):
            s.factor(nsw, "sync")
        same(("sync from A", nsw))
    for s in (a, b):   # warm start from the factor that is there, other values
        s.A.mul_(1.25)
    for nsw in (1, 2):
        for s in (a, b):
            s.factor(nsw, "sync", init="LU")
        same(("sync from LU", nsw))
    for s in (a, b):
        s.factor(1, "async")
    same("async from A")

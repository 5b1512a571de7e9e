"""Application sweeps taken two at a time (rows of at most three blocks a side, three sweeps or more)
against the sweeps one at a time, bit for bit.

Five mutually neighbouring cells appended to a system, not connected to it, have rows of four lower
and four upper blocks, so the same system then takes its sweeps one at a time; the rows of the
system itself have to come out the same."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SYSTEMS = [("chain", dict(n=1)), ("chain", dict(n=63)), ("chain", dict(n=65)), ("tri", dict(nx=1, ny=1)),
           ("tri", dict(nx=20, ny=13)), ("tri", dict(nx=17, ny=31, order="random")), ("quad", dict(nx=33, ny=16)),
           ("aniso", dict(nx=9, ny=60, order="line")), ("random", dict(n=9, deg=0.0)),
           ("clique3", dict())]


def system(kind, kw):
    from paper_1912_00539_amd import workloads as W
    if kind != "clique3":
        return W.case(kind, seed=2, **kw)
    a = np.array([0, 0, 1, 3]), np.array([1, 2, 2, 4])   # three mutual neighbours, a pair, a cell alone
    m = W.Mesh(6, *a, np.ones(4), "clique3", (6,))
    return W.assemble(m, W.natural_order(m), 3)


def with_five(c):
    from paper_1912_00539_amd import workloads as W
    i, j = np.triu_indices(5, 1)
    m = W.Mesh(5, i, j, np.ones(i.size), "clique5", (5,))
    d = W.assemble(m, W.natural_order(m), 4)
    return W.BSRCase(c.n + 5, np.concatenate([c.rowptr, c.rowptr[-1] + d.rowptr[1:]]).astype(np.int32),
                     np.concatenate([c.colidx, c.n + d.colidx]).astype(np.int32), np.concatenate([c.vals, d.vals]),
                     np.concatenate([c.b, d.b]), dict(c.meta))


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind,kw", SYSTEMS)
def test_pairs_equal_single_sweeps(kind, kw, prec):
    import torch
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = system(kind, kw)
    rows = np.repeat(np.arange(c.n), np.diff(c.rowptr))
    assert max(np.bincount(rows[c.colidx < rows], minlength=1)) <= 3 >= max(np.bincount(rows[c.colidx > rows], minlength=1))
    a, b = DeviceSystem(c, prec=prec), DeviceSystem(with_five(c), prec=prec)
    for s in (a, b):
        s.factor(2, "sync")
        s.work.fill_(255)   # the sweeps read nothing they have not written
    for nsw in (3, 4, 5, 6):
        za, zb = (torch.full_like(s.b, float("nan")) for s in (a, b))
        a.apply(a.b, za, nsw, "sync")
        b.apply(b.b, zb, nsw, "sync")
        assert torch.equal(za, zb[: 4 * c.n]), nsw
        a.apply(a.b, za.fill_(float("nan")), nsw, "async")   # pairs ping-pong in this mode too
        if nsw % 2 == 1:                                     # only pairs: the schedule is fixed
            assert torch.equal(za, zb[: 4 * c.n]), nsw

"""The chunked factor sweep on chains, in two launches (all rows at once, then the links along the
chain), where diagonal blocks are singular, need row exchanges or are huge: against the
workgroup-per-chunk runner bit for bit with its flags in both precisions, and in FP64 against the
oracle's chunked iteration. Rows have up to two, or three, blocks a side, and links at the edges of the
groups of rows that a quad fetches together."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_chunk_chains import lines

pytestmark = pytest.mark.gpu


def planted(kind, singular):
    c = lines(kind)
    rng = np.random.default_rng(17)
    rows = np.repeat(np.arange(c.n), np.diff(c.rowptr))
    d = np.flatnonzero(rows == c.colidx)
    c.vals = c.vals.copy()
    for i in rng.permutation(c.n)[:2 + c.n // 20]:
        c.vals[d[i]] = c.vals[d[i]][rng.permutation(4)]
    if singular is not None:
        c.vals[d[singular % c.n]] = 0.0
        c.vals[d[(singular + 5) % c.n]] *= 1e25
    return c


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind", ["chain", "grid", "lines3"])
@pytest.mark.parametrize("R,singular", [(1, 3), (2, None), (4, 4), (7, 11), (8, None), (9, 0), (16, 16), (40, -1)])
def test_links(kind, R, singular, prec):
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = planted(kind, singular)
    a, b = DeviceSystem(c, prec=prec), DeviceSystem(c, prec=prec)
    assert a.set_chunks(R, "rows")["runner"] == "rows" and b.set_chunks(R, "levels")["runner"] == "levels"

    def same(what):
        Xa, Da = a.factor_host()
        Xb, Db = b.factor_host()
        assert np.array_equal(Xa, Xb, equal_nan=True) and np.array_equal(Da, Db, equal_nan=True), what
        fa, fb = a.flags(clear=True), b.flags(clear=True)
        assert fa == fb, (what, fa, fb)
        return Xa, Da
    for s in (a, b):
        s.flags(clear=True)
    for nsw in (1, 2, 3):
        for s in (a, b):
            s.LU.fill_(float("nan"))    # the sweeps from A read neither
            s.Dinv.fill_(float("nan"))
            s.work.fill_(0)
            s.factor(nsw, "chunk_sync")
        X, D = same(("from A", nsw))
        if prec == "f64":
            Xo, Do, _ = oracle.factor_chunked(c.n, c.rowptr, c.colidx, c.vals, nsw, R)
            assert np.array_equal(X, Xo.reshape(X.shape), equal_nan=True), nsw
            assert np.array_equal(D, Do.reshape(D.shape), equal_nan=True), nsw
    for s in (a, b):
        s.A.mul_(1.5)
        s.factor(2, "chunk_sync", init="LU")
    same("from LU")
    # one asynchronous sweep from A: other chunks' operands are A's, as in a synchronous one (where
    # chunks are chains: the row runner, which chunks longer than a line take, reads inverses in place)
    rows = np.repeat(np.arange(c.n), np.diff(c.rowptr))
    if np.any((rows // R == c.colidx // R) & (np.abs(rows - c.colidx) > 1)):
        return
    a.factor(1, "chunk_sync")
    X, D = a.factor_host()
    a.LU.fill_(float("nan"))
    a.Dinv.fill_(float("nan"))
    a.factor(1, "chunk_async")
    Xa, Da = a.factor_host()
    assert np.array_equal(X, Xa, equal_nan=True) and np.array_equal(D, Da, equal_nan=True)

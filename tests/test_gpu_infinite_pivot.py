"""Factors where the last pivot of a diagonal block is infinite, as after an entry beyond the range of
single precision is rounded to it. Elimination divides by it, so the block has a finite inverse with a
row and column of zeros there and is not replaced: the flag word says NONFINITE (the block itself) and
not MODIFIED. Against the oracle's synchronous sweeps in FP64, bit for bit, and in FP32 within 1e-4
relative (sums of at most 3 products of blocks of condition below 100: 100 * 2^-24 * 16), and in both
precisions against the chunked sweeps with chunks of one row on a block diagonal pattern, where all
schedules are the same."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

MODIFIED, NONFINITE = 1, 2


def planted(kind, kw, value):
    from paper_1912_00539_amd import workloads as W
    c = W.case(kind, seed=6, **kw)
    rows = np.repeat(np.arange(c.n), np.diff(c.rowptr))
    d = np.flatnonzero(rows == c.colidx)
    c.vals = c.vals.copy()
    for i in (0, c.n // 2, c.n - 1):
        c.vals[d[i]][3, 3] = value
    return c


@pytest.mark.parametrize("prec,value", [("f64", np.inf), ("f32", np.inf), ("f32", 1e200), ("f32", -1e200)])
@pytest.mark.parametrize("kind,kw", [("random", dict(n=70, deg=0.0)), ("tri", dict(nx=9, ny=7)),
                                     ("tri", dict(nx=17, ny=15, order="random")), ("random", dict(n=90, deg=7.0))])
def test_infinite_last_pivot(kind, kw, prec, value):
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = planted(kind, kw, value)
    vals = c.vals if prec == "f64" else c.vals.astype(np.float32).astype(np.float64)
    s = DeviceSystem(c, prec=prec)

    def check(Xo, Do, what):
        X, D = s.factor_host()
        Xo, Do = Xo.reshape(X.shape), Do.reshape(D.shape)
        assert np.isfinite(Do).all()
        assert s.flags(clear=True) == NONFINITE, what
        if prec == "f64":
            assert np.array_equal(X, Xo) and np.array_equal(D, Do), what
        else:
            fin = np.isfinite(Xo)
            assert np.array_equal(X[~fin], Xo[~fin]), what
            for got, ref in ((X[fin], Xo[fin]), (D, Do)):
                assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max(), what

    s.flags(clear=True)
    with np.errstate(all="ignore"):
        for nsw in (1, 2):
            Xo, Do, flags = oracle.factor_sync(c.n, c.rowptr, c.colidx, vals, nsw)
            assert flags == NONFINITE
            s.factor(nsw, "sync")
            check(Xo, Do, ("sync", nsw))
        if kind == "random" and kw["deg"] == 0.0:
            Xo, Do, _ = oracle.factor_sync(c.n, c.rowptr, c.colidx, vals, 1)
            s.factor(1, "async")
            check(Xo, Do, "async")
            X, D = s.factor_host()
            for runner in ("rows", "levels"):
                s.set_chunks(1, runner)
                s.factor(1, "chunk_sync")
                check(Xo, Do, runner)
                assert np.array_equal(s.factor_host()[1], D), runner

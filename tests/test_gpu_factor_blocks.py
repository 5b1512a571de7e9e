"""The synchronous factor sweep with a quad per block (patterns with update sets off the diagonal, or
rows of more than three lower or upper blocks) against the oracle on structurally unsymmetric patterns
around the tile of 64 blocks and over several slabs: in FP64 bit for bit, with its flags, where diagonal
blocks are singular or need row exchanges too. In FP32, on nonsingular ones, within
u (4 p + 16 c) per sweep: u = 2^-24, p update pairs of four products each, and an inverse whose error
grows with the condition c of the worst diagonal block."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# (cells, mean neighbours, share of the off-diagonal blocks that stays)
PATTERNS = [(9, 8.0, 1.0), (16, 8.0, 0.5), (63, 7.0, 0.7), (64, 9.0, 1.0), (65, 12.0, 0.8), (257, 6.0, 0.6),
            (1024, 5.0, 0.9), (20000, 6.0, 0.7)]


def unsymmetric(n, deg, share, singular):
    from paper_1912_00539_amd import workloads as W
    from paper_1912_00539_amd.workloads import BSRCase
    c = W.case("random", seed=31, n=n, deg=deg)
    rng = np.random.default_rng(7)
    rows = np.repeat(np.arange(n), np.diff(c.rowptr))
    diag = rows == c.colidx
    keep = diag | (rng.random(len(rows)) < share)
    vals = c.vals.copy()
    d = np.flatnonzero(diag)
    for i in rng.permutation(n)[:2 + n // 30]:      # blocks that need row exchanges
        vals[d[i]] = vals[d[i]][rng.permutation(4)]
    if singular:
        vals[d[n - 1]] = 0.0                        # its inverse is asked for by no lower block
        vals[d[n // 2]] = 0.0
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=n))]).astype(np.int32)
    return BSRCase(n, rp, c.colidx[keep].astype(np.int32), vals[keep], c.b, dict(c.meta))


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,deg,share", PATTERNS)
def test_block_form(n, deg, share, prec):
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = unsymmetric(n, deg, share, prec == "f64")
    s = DeviceSystem(c, prec=prec)
    p = int(np.diff(oracle.pairs(c.n, c.rowptr, c.colidx)[0]).max())
    s.flags(clear=True)

    def check(nsw, X0, what):
        X, D = s.factor_host()
        vals = s.A.cpu().numpy().reshape(c.vals.shape)
        Xo, Do, flags = oracle.factor_sync(c.n, c.rowptr, c.colidx, vals, nsw, X0=X0)
        Xo, Do = Xo.reshape(X.shape), Do.reshape(D.shape)
        if prec == "f64":
            assert np.array_equal(X, Xo, equal_nan=True) and np.array_equal(D, Do, equal_nan=True), what
            assert s.flags(clear=True) == flags, what
            return X
        cond = np.linalg.cond(Do.astype(np.float64)).max()
        tol = nsw * 2.0 ** -24 * (4 * p + 16 * cond)
        for got, ref in ((X, Xo), (D, Do)):
            assert np.abs(got - ref).max() <= tol * np.abs(ref).max(), (what, cond)
        assert s.flags(clear=True) == 0, what
        return X.astype(np.float64)

    for nsw in (1, 2, 3):
        s.factor(nsw, "sync")
        X = check(nsw, None, ("from A", nsw))
    s.A.mul_(1.25)
    for nsw in (1, 2):
        s.factor(nsw, "sync", init="LU")
        X = check(nsw, X, ("from LU", nsw))

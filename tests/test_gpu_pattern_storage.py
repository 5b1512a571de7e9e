"""Where abilu_build_pattern keeps the records of its analysis: in its own scratch where they fit, in an
allocation of their own on large patterns, and after the symmetry is known on unsymmetric patterns whose
update sets are as many as their lower blocks. Against the oracle's synchronous factor and application in
FP64, bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def triples(copies):
    """Three rows, {0, 1, 2}, {1}, {0, 1, 2}, over and over: two lower blocks and two pairs each, one pair
    off the diagonal, (0, 1) without (1, 0)."""
    from paper_1912_00539_amd.workloads import BSRCase
    rng = np.random.default_rng(copies)
    n = 3 * copies
    col = (np.array([0, 1, 2, 1, 0, 1, 2])[None, :] + 3 * np.arange(copies)[:, None]).reshape(-1)
    rp = np.concatenate([[0], np.cumsum(np.tile([3, 1, 3], copies))])
    vals = 0.2 * rng.standard_normal((len(col), 4, 4))
    vals[np.repeat(np.arange(n), np.diff(rp)) == col] += 4.0 * np.eye(4)
    return BSRCase(n, rp.astype(np.int32), col.astype(np.int32), vals, rng.standard_normal(4 * n), dict(kind="triples"))


def case(kind, size):
    from paper_1912_00539_amd import workloads as W
    if kind == "triples":
        return triples(size)
    if kind == "random":
        return W.case("random", seed=8, n=size, deg=6.0)
    return W.case(kind, seed=8, nx=size, ny=max(1, 9 * size // 10))


@pytest.mark.parametrize("kind,size", [("triples", 1), ("triples", 50), ("triples", 7001), ("random", 300), ("quad", 1),
                                       ("quad", 40), ("tri", 40), ("quad", 1000)])
def test_records_wherever_they_are_kept(kind, size):
    import torch
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = case(kind, size)
    s = DeviceSystem(c, prec="f64", restart=0)
    junk = torch.full((1 << 22,), -1, dtype=torch.int32, device="cuda")   # takes over what the build gave back
    s.factor(2, "sync")
    X, D, _ = oracle.factor_sync(c.n, c.rowptr, c.colidx, c.vals, 2)
    got, Dg = s.factor_host()
    assert np.array_equal(got, X.reshape(got.shape)) and np.array_equal(Dg, D.reshape(Dg.shape))
    for nsw in (3, 4):
        z = torch.full_like(s.b, float("nan"))
        s.apply(s.b, z, nsw, "sync")
        assert np.array_equal(z.cpu().numpy(), oracle.apply_sync(c.n, c.rowptr, c.colidx, X, D, c.b, nsw)), nsw
    assert int(junk.sum()) == -(1 << 22)

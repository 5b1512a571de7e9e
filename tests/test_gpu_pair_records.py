"""Pairs of application sweeps on rows of at most two blocks a side, whose indices come from the
pattern's records, on structurally unsymmetric patterns (rows with none, one or two blocks on either
side, in all combinations with their neighbours') against the oracle's synchronous sweeps in FP64,
bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def banded(n, far, share, seed):
    from paper_1912_00539_amd.workloads import BSRCase
    rng = np.random.default_rng(seed)
    ptr, col = [0], []
    for i in range(n):
        near = [j for j in sorted({i - far, i - 1, i + 1, i + far}) if 0 <= j < n and j != i and rng.random() < share]
        col += sorted(near + [i])
        ptr.append(len(col))
    col = np.array(col, np.int32)
    rows = np.repeat(np.arange(n), np.diff(ptr))
    vals = 0.2 * rng.standard_normal((len(col), 4, 4))
    vals[rows == col] += 4.0 * np.eye(4)
    return BSRCase(n, np.array(ptr, np.int32), col, vals, rng.standard_normal(4 * n), dict(kind="banded"))


@pytest.mark.parametrize("n,far,share", [(1, 2, 1.0), (2, 2, 1.0), (5, 2, 0.6), (63, 7, 0.7), (64, 3, 1.0),
                                         (65, 64, 0.8), (300, 17, 0.5), (1500, 40, 0.8)])
def test_records(n, far, share):
    import torch
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = banded(n, far, share, 5 + n)
    s = DeviceSystem(c, prec="f64")
    X, D, _ = oracle.factor_sync(c.n, c.rowptr, c.colidx, c.vals, 2)
    s.factor(2, "sync")
    for nsw in (3, 4, 5):
        z = torch.full_like(s.b, float("nan"))
        s.apply(s.b, z, nsw, "sync")
        assert np.array_equal(z.cpu().numpy(), oracle.apply_sync(c.n, c.rowptr, c.colidx, X, D, c.b, nsw)), nsw

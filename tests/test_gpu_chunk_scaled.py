"""Chunked applications inside FGMRES, whose right-hand sides are unnormalised basis vectors with a factor,
in every runner: with a block diagonal matrix and its exact factor the preconditioned operator is the
identity, so FGMRES ends after one step with the solution, whatever the size of b. And outside of it the
application of a scaled vector is the scaled application."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RUNNERS = [(3, "rows"), (16, "rows"), (40, "rows"), (16, "levels")]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("R,runner", RUNNERS)
@pytest.mark.parametrize("kind,kw", [("aniso", dict(nx=30, ny=45, order="line")), ("tri", dict(nx=20, ny=21)),
                                     ("random", dict(n=300, deg=7.0))])
def test_factor_on_the_right_hand_side(kind, kw, R, runner, prec):
    import torch
    from paper_1912_00539_amd import workloads as W
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = W.case(kind, seed=9, **kw)
    s = DeviceSystem(c, prec=prec)
    s.set_chunks(R, runner)
    s.factor(2, "chunk_sync")
    z, y = torch.empty_like(s.b), torch.empty_like(s.b)
    for nsw in (1, 2):
        s.apply(s.b, z, nsw, "chunk_sync")
        s.apply(s.b * 1024.0, y, nsw, "chunk_sync")   # powers of two change no rounding
        assert torch.equal(y, z * 1024.0), nsw
    rows = np.repeat(np.arange(c.n), np.diff(c.rowptr))
    c.vals = np.where((rows == c.colidx)[:, None, None], c.vals, 0.0)
    for scale in (1.0, 1e-6, 1e6):
        s.load_values(c.vals, c.b * scale)
        s.factor(1, "chunk_sync")
        st, r = s.solve(apply_sweeps=2, mode="chunk_sync", rtol=1e-4, maxit=20)
        assert st == 0 and r["iters"] == 1, (scale, r)

"""FGMRES's host loop: the polled status and the applications begun ahead of it, at a size of each
look-ahead (two sweeps, one, none), where a solve ends in each of the ways it can end."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(33, 31), (260, 251), (701, 601)]   # cells: 1,023; 65,260; 421,301


def system(nx, ny, prec="f64", restart=5):
    from paper_1912_00539_amd import workloads as W
    from paper_1912_00539_amd.runtime import DeviceSystem
    s = DeviceSystem(W.case("quad", seed=1, nx=nx, ny=ny, s=0.5), prec=prec, restart=restart)
    s.factor(2, "sync")
    return s


@pytest.mark.parametrize("nx,ny", SIZES)
def test_ends_before_the_first_cycle(nx, ny):
    """Converged at the start, no iteration allowed, b = 0: x is the zero guess although no cycle wrote it."""
    from paper_1912_00539_amd import abilu as L
    s = system(nx, ny)
    for kw, st, conv in ((dict(rtol=1.0), L.ABILU_OK, 1), (dict(rtol=1e-8, maxit=0), L.ABILU_WARN_NOCONV, 0)):
        s.x.fill_(float("nan"))
        got, r = s.solve(apply_sweeps=3, mode="sync", **kw)
        assert (got, r["iters"], r["converged"], r["rel_true_residual"]) == (st, 0, conv, 1.0)
        assert not s.x.any()
    s.b.zero_()
    s.x.fill_(float("nan"))
    got, r = s.solve(apply_sweeps=3, mode="async", rtol=1e-8)
    assert (got, r["iters"], r["converged"]) == (L.ABILU_OK, 0, 1) and not s.x.any()
    s.b.fill_(float("nan"))
    got, r = s.solve(apply_sweeps=3, mode="async", rtol=1e-8)
    assert got == L.ABILU_ENONFINITE and r["iters"] == 0 and not s.x.any()


@pytest.mark.parametrize("nx,ny", SIZES)
@pytest.mark.parametrize("nsw", [0, 1, 2, 3])
def test_restarts_and_both_initial_guesses(nx, ny, nsw):
    """Restarts of two steps to 1e-10: the true residual the solve reports is the one of its x, and an
    explicit zero guess (one SpMV and a read of x more) takes the same steps to the same x."""
    import torch
    s = system(nx, ny)
    st, r = s.solve(apply_sweeps=nsw, mode="sync", rtol=1e-10, maxit=400, restart=2)
    x = s.x.clone()
    y = torch.empty_like(x)
    s.spmv(x, y)
    true = float((s.b - y).norm() / s.b.norm())
    assert st == 0 and r["restarts"] > 1 and true <= 1e-10
    assert abs(true - r["rel_true_residual"]) <= 1e-14
    st, r2 = s.solve(apply_sweeps=nsw, mode="sync", rtol=1e-10, maxit=400, restart=2, x0=torch.zeros_like(x))
    assert (r2["iters"], r2["restarts"], r2["reorth"]) == (r["iters"], r["restarts"], r["reorth"])
    assert float((s.x - x).norm()) <= 1e-12 * float(x.norm())


def test_refused_while_the_stream_is_captured():
    import torch
    from paper_1912_00539_amd import abilu as L
    s = system(*SIZES[0])
    s.solve(apply_sweeps=3, mode="sync", rtol=1e-8)
    x = s.x.clone()
    g = torch.cuda.CUDAGraph()
    z = torch.zeros(8, device="cuda")
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        z += 1
        with pytest.raises(L.AbiluError) as e:
            s.solve(apply_sweeps=3, mode="sync", rtol=1e-8)
        assert e.value.status == L.ABILU_EDEVICE
    g.replay()
    torch.cuda.synchronize()
    assert float(z.sum()) == 8.0 and torch.equal(s.x, x)

"""What the in-place chunked mode is for: rows of other chunks are read as they are in memory, so on lines of
cells whose chunks run side by side a sweep sees values of the same sweep and converges faster than the
synchronous one. On meshes of chains: the distance of the application from the triangular solves, and the
residual of the factor equations after its second sweep. The margins are a fifth and less of what the
in-place sweeps gain (three sweeps 2.5 and 1.8 times, six 80 and 8 times; second factor sweep 300 and 25
times), since the gain depends on scheduling."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def mesh(kind):
    from paper_1912_00539_amd import workloads as W
    if kind == "aniso":
        return W.case("aniso", seed=1, nx=1000, ny=500, order="line", shift="cfl", cfl=100.0), 16, (0.75, 0.1, 0.05)
    k, nz = 50, 60
    q = np.arange(k * k * nz).reshape(nz, k, k)
    fa = np.concatenate([q[:-1].ravel(), q[:, :-1].ravel(), q[:, :, :-1].ravel()])
    fb = np.concatenate([q[1:].ravel(), q[:, 1:].ravel(), q[:, :, 1:].ravel()])
    m = W.Mesh(q.size, fa, fb, np.ones(fa.size), "hexahedra", (k, k, nz))
    return W.assemble(m, W.natural_order(m), 3, "cfl", cfl=100.0), 48, (0.85, 0.5, 0.4)


@pytest.mark.parametrize("kind", ["aniso", "hexahedra"])
def test_in_place_sweeps_converge_faster(kind):
    import torch
    from paper_1912_00539_amd.runtime import DeviceSystem
    c, R, (three, six, second) = mesh(kind)
    s = DeviceSystem(c, prec="f64", restart=0)
    s.factor(3, "sync")
    exact, z = torch.empty_like(s.b), torch.empty_like(s.b)
    s.apply(s.b, exact, 60, "sync")
    assert s.set_chunks(R, "rows")["runner"] == "rows"

    def away(nsw, mode):
        s.apply(s.b, z, nsw, mode)
        return float((z - exact).norm() / exact.norm())
    for nsw, margin in ((3, three), (6, six)):
        a, b = away(nsw, "chunk_async"), away(nsw, "chunk_sync")
        assert a <= margin * b, (nsw, a, b)
    s.set_chunks(16, "rows")

    def residual(mode):
        s.factor(2, mode)
        return s.ilu_residual()
    a, b = residual("chunk_async"), residual("chunk_sync")
    assert a <= second * b, (a, b)

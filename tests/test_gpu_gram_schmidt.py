"""FGMRES's fused Gram-Schmidt kernels at the sizes where their forms change: the vector tile (edges
of 1,024 elements), the folded reductions (at most 512 tiles) and the register forms of the update
with the second pass's dots (4, 8, 16, 32 basis vectors, then any number).

Without a preconditioner (0 apply sweeps) FGMRES is GMRES on A, whose residual after k steps is the
least-squares minimum over the Krylov space of b. The reference builds that space in NumPy with
Householder QR and takes the minimum; with orthogonality at rounding level the two agree to
k^2 * 1e-15 * cond, far inside 1e-9."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def krylov_minimum(c, k):
    """min ||b - A x|| / ||b|| over x in span{b, A b, ..., A^{k-1} b}, by Arnoldi with full QR."""
    import scipy.sparse as sp
    A = sp.bsr_matrix((c.vals, c.colidx, c.rowptr), shape=(4 * c.n, 4 * c.n))
    Q = np.zeros((4 * c.n, k + 1))
    H = np.zeros((k + 1, k))
    Q[:, 0] = c.b / np.linalg.norm(c.b)
    for j in range(k):
        w = A @ Q[:, j]
        for _ in range(3):
            h = Q[:, :j + 1].T @ w
            w -= Q[:, :j + 1] @ h
            H[:j + 1, j] += h
        H[j + 1, j] = np.linalg.norm(w)
        Q[:, j + 1] = w / H[j + 1, j]
    e = np.zeros(k + 1)
    e[0] = 1.0
    y = np.linalg.lstsq(H, e, rcond=None)[0]
    return np.linalg.norm(e - H @ y)


# cells: one tile less one cell, one tile, one more (k around each register form and past the last);
# the largest folded system, the next (one k per form)
CASES = [(nx, ny, k) for nx, ny in ((5, 51), (16, 16), (257, 1)) for k in (1, 4, 5, 8, 9, 16, 17, 32, 33, 40)]
CASES += [(nx, ny, k) for nx, ny in ((256, 512), (11917, 11)) for k in (1, 5, 9, 17, 33)]


@pytest.mark.parametrize("nx,ny,k", CASES)
def test_gmres_residual_is_the_krylov_minimum(nx, ny, k):
    from paper_1912_00539_amd import abilu as L
    from paper_1912_00539_amd import workloads as W
    from paper_1912_00539_amd.runtime import DeviceSystem
    c = W.case("quad", seed=3, nx=nx, ny=ny, s=1.0)
    s = DeviceSystem(c, prec="f64", restart=k)
    st, r = s.solve(apply_sweeps=0, mode="sync", rtol=0.0, maxit=k)
    assert r["iters"] == k and st == L.ABILU_WARN_NOCONV, r
    ref = krylov_minimum(c, k)
    assert abs(r["rel_true_residual"] - ref) <= 1e-9 * ref + 1e-13, (r, ref)
    assert abs(r["rel_estimate"] - ref) <= 1e-9 * ref + 1e-13, (r, ref)

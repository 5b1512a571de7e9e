"""The asynchronous first factor sweep from A on a pattern with long rows whose matrix is larger than the
last-level cache (the launch that bounds the workgroups of a compute unit). With zero values below the
diagonal L = 0 and U = A whatever the schedule, so the result equals the synchronous sweep's, and the
inverses those of A's diagonal blocks (of condition below 10: 16 * 10 rounding errors)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_first_sweep(prec):
    import torch
    from paper_1912_00539_amd import abilu as L
    n, w = 110000, 10      # rows of 21 blocks, columns i - 10 .. i + 10: 2.3 million blocks, 296 MB
    col = (torch.arange(n, device="cuda")[:, None] + torch.arange(-w, w + 1, device="cuda")[None, :])
    keep = (col >= 0) & (col < n)
    row = torch.arange(n, device="cuda")[:, None].expand_as(col)[keep]
    colidx = col[keep].to(torch.int32)
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(keep.sum(1), 0)
    z = colidx.numel()
    assert z >= 18 * n and 128 * z > 256 << 20
    g = torch.Generator(device="cuda").manual_seed(4)
    A = torch.zeros(z, 4, 4, dtype=torch.float64, device="cuda")
    diag = (row == colidx.long()).nonzero().reshape(-1)
    A[diag] = torch.rand(n, 4, 4, generator=g, dtype=torch.float64, device="cuda") + 8.0 * torch.eye(4, device="cuda").double()
    upper = (row < colidx.long()).nonzero().reshape(-1)
    A[upper] = torch.rand(upper.numel(), 4, 4, generator=g, dtype=torch.float64, device="cuda")
    p = L.abilu_build_pattern(n, rowptr, colidx)   # no lower values: L = 0, U = A
    dt = torch.float64 if prec == "f64" else torch.float32
    work = torch.zeros(L.abilu_workspace_bytes(p, prec, 0), dtype=torch.uint8, device="cuda")
    out = []
    for mode in ("async", "sync"):
        LU = torch.full((16 * z,), float("nan"), dtype=dt, device="cuda")
        D = torch.full((16 * n,), float("nan"), dtype=dt, device="cuda")
        L.abilu_factor(p, A.reshape(-1), LU, D, prec, 1, mode, work)
        out.append((LU, D))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert torch.isfinite(out[0][0]).all() and torch.isfinite(out[0][1]).all()
    inv = torch.linalg.inv(A[diag])
    assert float((out[0][1].reshape(n, 4, 4).double() - inv).abs().max()) < (1e-14 if prec == "f64" else 1e-5)

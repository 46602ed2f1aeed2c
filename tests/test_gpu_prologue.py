"""The passes before a product (column sums, finiteness, column maxima, packs)
at the edges of their work split: a workgroup of the prologue owns at least 128
consecutive points and there are at most 128 of them, a pack workgroup takes
128 points, a bfloat16 row is read 16 bytes at a time only where it is aligned.

Each size is checked through the product against the float64 oracle (far from
the origin, so a wrong mean shows), and with one non-finite value in the last
point of the row or of the column set, which every output must report.
"""
import numpy as np
import pytest
import torch

from gpu_util import TOL_BF16, TOL_F32, case, device, rel_fro, to_np
from oracle import kernel as ok
from paper_2609_38198_amd import _lib as fd

pytestmark = pytest.mark.gpu


def _points(n, d, pad, dtype, seed):
    """n x d points in rows of d + pad elements, and their float64 values."""
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(n, d + pad, generator=g) * 0.3
    if dtype == torch.float32:
        x += 20.0  # centred inside; bfloat16 data is taken as given
    x = x.to(dtype).to(device())[:, :d]
    return x, x.double().cpu().numpy()


@pytest.mark.parametrize("n, d, pad, b", [(1, 3, 0, 2), (127, 1, 0, 3), (128, 13, 1, 1),
                                          (129, 30, 0, 5), (16383, 8, 0, 4), (16384, 31, 2, 16),
                                          (16513, 62, 0, 17), (20000, 64, 0, 64)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_product_at_the_edges_of_the_prologue(n, d, pad, b, dtype):
    case(f"prologue n={n} d={d} pad={pad} b={b} {dtype}")
    tol = TOL_F32 if dtype == torch.float32 else TOL_BF16
    x, x64 = _points(n, d, pad, dtype, n + d)
    V = torch.randn(n, b, generator=torch.Generator().manual_seed(7)).to(device())
    beta = 1.0 / d
    rows = np.unique(np.linspace(0, n - 1, 40).astype(int))
    Y = to_np(fd.fd_kernel_matmul(x, None, beta, V))[rows]
    ref = ok.kernel_matmul(x64[rows], x64, beta, to_np(V))
    assert rel_fro(Y, ref) <= tol
    # rows from a set of their own, of another size
    xr, xr64 = _points(n // 3 + 1, d, pad, dtype, n + 1)
    Y = to_np(fd.fd_kernel_matmul(xr, x, beta, V))
    pick = np.unique(np.linspace(0, len(xr64) - 1, 40).astype(int))
    assert rel_fro(Y[pick], ok.kernel_matmul(xr64[pick], x64, beta, to_np(V))) <= tol
    bad = x.clone()
    bad[n - 1, d - 1] = float("inf")
    assert np.isnan(to_np(fd.fd_kernel_matmul(bad, None, beta, V))).all()
    badr = xr.clone()
    badr[-1, 0] = float("nan")
    if badr.stride(0) == x.contiguous().stride(0):
        assert np.isnan(to_np(fd.fd_kernel_matmul(badr, x.contiguous(), beta, V))).all()
    deg = fd.fd_degree(bad, beta)
    for t in (deg.q, deg.d, deg.s, deg.s_off):
        assert torch.isnan(t).all()

"""The passes before a product (column sums, finiteness, column maxima, packs)
at the edges of their work split: a workgroup of the prologue owns at least 128
consecutive points and there are at most 128 of them, above 2^15 points with
3 * 2^18 values (column sums: 2^22) up to 1,024 and a second launch that adds their results, a pack workgroup takes
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


@pytest.mark.parametrize("n, d, b", [(32768, 33, 33), (32769, 24, 1), (32769, 23, 23),
                                     (32769, 4, 24), (32769, 24, 4), (150001, 7, 7),
                                     (131072, 31, 2), (131072, 32, 2),
                                     (262144, 4, 1), (262145, 4, 64), (300001, 64, 3)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_product_against_many_points(n, d, b, dtype):
    """Both sides of the lines of the second launch, and more points than its
    workgroups take 256 each; the columns of V are of very different size, the
    largest value of one in the last row."""
    case(f"prologue, many points n={n} d={d} b={b} {dtype}")
    tol = TOL_F32 if dtype == torch.float32 else TOL_BF16
    x, x64 = _points(n, d, 0, dtype, n + d)
    xr, xr64 = _points(40, d, 0, dtype, n + 1)
    # of one sign: sums over many points do not cancel
    V = torch.rand(n, b, generator=torch.Generator().manual_seed(7)) + 0.5
    V *= torch.exp2(torch.arange(b) - 20.0)
    V[n - 1, b // 2] *= 1e4
    V = V.to(device())
    beta = 1.0 / d
    Y = to_np(fd.fd_kernel_matmul(xr, x, beta, V))
    ref = ok.kernel_matmul(xr64, x64, beta, to_np(V))
    err = max(rel_fro(Y[:, c], ref[:, c]) for c in range(b))
    assert err <= tol
    for where, value in ((n - 1, float("inf")), (n // 2, float("nan"))):
        bad = x.clone()
        bad[where, d - 1] = value
        assert np.isnan(to_np(fd.fd_kernel_matmul(xr, bad, beta, V))).all()
        W = V.clone()
        W[where, 0] = value
        assert not np.isfinite(to_np(fd.fd_kernel_matmul(xr, x, beta, W))[:, 0]).any()

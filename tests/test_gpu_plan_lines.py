"""Products and row sums on both sides of the lines of their work split: at
most 2^28 pairs take four row tiles per wave, one 16-column block at D <= 12
above takes eight; at most 3 * 2^27 pairs are split for one resident round of
workgroups; a symmetric row sum of at most 48 blocks of 512 points for one
resident round, from 64 on by whole blocks.

Tolerances are those of the arithmetic whatever the split: a split only says
where a row's sum is cut, and its parts are added in float64.
"""
import numpy as np
import pytest
import torch

from gpu_util import TOL_BF16, TOL_F32, case, device, rel_fro, to_np
from oracle import kernel as ok
from paper_2609_38198_amd import _lib as fd

pytestmark = pytest.mark.gpu


def _points(n, d, dtype):
    x = torch.randn(n, d, generator=torch.Generator().manual_seed(n + d)) * 0.5
    x = x.to(dtype).to(device())
    return x, x.double().cpu().numpy()


@pytest.mark.parametrize("nr, nc", [(1024, 1 << 18), (1024, (1 << 18) + 1), (1024, 3 << 17),
                                    (1025, 3 << 17)])
@pytest.mark.parametrize("d, b", [(12, 16), (5, 3), (12, 17)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_product_at_the_lines(nr, nc, d, b, dtype):
    case(f"plan lines nr={nr} nc={nc} d={d} b={b} {dtype}")
    xr, xr64 = _points(nr, d, dtype)
    xc, xc64 = _points(nc, d, dtype)
    V = torch.randn(nc, b, generator=torch.Generator().manual_seed(7)).to(device())
    beta = float(np.float32(1.0 / d))
    rows = np.unique(np.linspace(0, nr - 1, 20).astype(int))
    Y = fd.fd_kernel_matmul(xr, xc, beta, V)
    ref = ok.kernel_matmul(xr64[rows], xc64, beta, to_np(V))
    assert rel_fro(to_np(Y)[rows], ref) <= (TOL_F32 if dtype == torch.float32 else TOL_BF16)
    assert torch.equal(Y, fd.fd_kernel_matmul(xr, xc, beta, V))


@pytest.mark.parametrize("n", [17 * 512, 48 * 512, 48 * 512 + 1, 63 * 512, 63 * 512 + 1])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_row_sums_at_the_lines(n, dtype):
    case(f"plan lines n={n} {dtype}")
    d = 12
    x, x64 = _points(n, d, dtype)
    beta = float(np.float32(1.0 / d))
    deg = fd.fd_degree(x, beta, 0.5)
    rows = np.unique(np.linspace(0, n - 1, 40).astype(int))
    assert rel_fro(to_np(deg.q)[rows],
                   ok.kernel_matmul(x64[rows], x64, beta, np.ones((n, 1)))[:, 0]) <= TOL_F32
    w = to_np(deg.q) ** -0.5
    dd = w[rows] * ok.kernel_matmul(x64[rows], x64, beta, w[:, None])[:, 0]
    assert rel_fro(to_np(deg.d)[rows], dd) <= TOL_F32


def _square_error(n, d, b, seed):
    """Relative Frobenius error of a square product against float64 (all rows)."""
    g = torch.Generator(device=device()).manual_seed(seed)
    x = torch.randn(n, d, generator=g, device=device()) * 0.3
    V = torch.randn(n, b, generator=g, device=device())
    beta = float(np.float32(4.0 / d))
    Y = fd.fd_kernel_matmul(x, None, beta, V).double()
    xd, num, den = x.double(), 0.0, 0.0
    r, xt = xd.square().sum(1), xd.T.contiguous()
    for i in range(0, n, 2000):
        a = xd[i:i + 2000]
        h = (r + a.square().sum(1, keepdim=True) - 2 * a @ xt).clamp_(min=0)
        m = torch.arange(len(a), device=device())
        h[m, m + i] = 0
        ref = (-beta * h).exp() @ V.double()
        num += float((Y[i:i + 2000] - ref).square().sum())
        den += float(ref.square().sum())
    return (num / den) ** 0.5


@pytest.mark.parametrize("n, d, b, bound", [(5000, 12, 16, 7.48e-7), (8000, 30, 32, 9.38e-7),
                                            (16000, 12, 32, 8.16e-7), (16000, 30, 16, 9.79e-7)])
def test_one_round_keeps_the_error_of_many_splits(n, d, b, bound):
    """Mean over six seeds of inputs, which are the same everywhere and so are the
    bits of the product; `bound` is the mean with the columns split for 2,048
    workgroups (7.451, 9.334, 8.122 and 9.738e-7) and half a percent."""
    case(f"one-round error n={n} d={d} b={b}")
    assert np.mean([_square_error(n, d, b, seed) for seed in range(6)]) <= bound

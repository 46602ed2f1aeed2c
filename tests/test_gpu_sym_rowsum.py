"""The symmetric row sums over their two other users: bfloat16 points and a
single right-hand side.

They pair blocks of 512 points, each unordered pair of blocks evaluated once, so
the sizes here are one block and its edges, an even and an odd number of
blocks, and 64 blocks and more, where column splits become whole blocks.
Tolerances: the vectors of fd_degree and one float32 column to 1e-5 (the
stated tolerance of float32 arithmetic); bfloat16 points enter exactly, so
their sums keep that bar.  One column's sums along the columns are fixed point
with 53 fractional bits against the largest weight, for columns whose span
leaves 2^-18 of the smallest weight at this size.
"""
import numpy as np
import pytest
import torch

from gpu_util import TOL_F32, case, device, rel_fro, to_np
from oracle import kernel as ok
from oracle import normalise as on
from paper_2609_38198_amd import _lib as fd

pytestmark = pytest.mark.gpu

SIZES = [(5, 3), (511, 12), (512, 40), (513, 64), (1024, 7), (1536, 33), (2049, 64), (5000, 30)]


def _points(n, d, dtype):
    x = torch.randn(n, d, generator=torch.Generator().manual_seed(n + d)) * 0.5
    x = x.to(dtype).to(device())
    return x, x.double().cpu().numpy()


@pytest.mark.parametrize("n, d", SIZES)
@pytest.mark.parametrize("alpha", [0.0, 0.5])
def test_bfloat16_normalisation(n, d, alpha):
    case(f"degree bf16 n={n} d={d} alpha={alpha}")
    x, x64 = _points(n, d, torch.bfloat16)
    deg = fd.fd_degree(x, 1.0 / d, alpha)
    ref = on.normalise(x64, float(np.float32(1.0 / d)), alpha)
    for name in ("q", "d", "s"):
        assert rel_fro(to_np(getattr(deg, name)), getattr(ref, name)) <= TOL_F32
    assert abs(float(to_np(deg.s_off)[0]) - ref.s_off) <= TOL_F32 * float(ref.q.sum())


def test_bfloat16_normalisation_with_whole_block_splits_and_dyadic_levels():
    n, d = 40000, 20
    case(f"degree bf16 n={n} d={d}, dyadic")
    x, x64 = _points(n, d, torch.bfloat16)
    lev = fd.fd_degree_dyadic(x, 0.25 / d, 3, 0.5)
    again = fd.fd_degree_dyadic(x, 0.25 / d, 3, 0.5)
    assert torch.equal(lev.q, again.q) and torch.equal(lev.s, again.s)
    rows = np.linspace(0, n - 1, 50).astype(int)
    beta0 = float(np.float32(0.25 / d))
    for l in range(3):
        beta = beta0 * 2 ** l
        q = ok.kernel_matmul(x64[rows], x64, beta, np.ones((n, 1)))[:, 0]
        assert rel_fro(to_np(lev.q)[l][rows], q) <= TOL_F32
        w = to_np(lev.q)[l] ** -0.5
        dd = w[rows] * ok.kernel_matmul(x64[rows], x64, beta, w[:, None])[:, 0]
        assert rel_fro(to_np(lev.d)[l][rows], dd) <= TOL_F32


@pytest.mark.parametrize("n", [700, 2048, 6800])
@pytest.mark.parametrize("beta", [37.0, 1234.5, 7.7e4])
def test_bfloat16_points_that_coincide_far_from_the_origin(n, beta):
    """64 places on a grid of 4 (norms up to 1e4, exact in float32) at beta |x|^2
    far beyond any budget: a kernel value is 1 within a place, and at most
    exp(-16 beta) = 0 in float32 between them, so that the sums are counts."""
    case(f"coincident bf16 points n={n} beta={beta}")
    base = 4.0 * torch.randint(-8, 9, (64, 16), generator=torch.Generator().manual_seed(3))
    place = torch.arange(n) % 64
    assert len(torch.unique(base, dim=0)) == 64
    x = base[place].to(torch.bfloat16).to(device())
    count = torch.bincount(place, minlength=64)[place].double().numpy()
    deg = fd.fd_degree(x, beta, 0.5)
    assert np.array_equal(to_np(deg.q), count)
    assert rel_fro(to_np(deg.d), np.ones(n)) <= TOL_F32
    Y = fd.fd_kernel_matmul(x, None, beta, torch.ones(n, 1, device=device()))
    assert np.array_equal(to_np(Y)[:, 0], count)


# a single column takes the symmetric sums from 6,144 points on
COLUMN_SIZES = [(6143, 12), (6144, 40), (6145, 3), (6657, 64), (7001, 30), (40001, 12)]


@pytest.mark.parametrize("n, d", SIZES + COLUMN_SIZES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_one_column(n, d, dtype):
    case(f"one column n={n} d={d} {dtype}")
    x, x64 = _points(n, d, dtype)
    g = torch.Generator().manual_seed(3)
    v = torch.randn(n, 1, generator=g) * torch.exp2(16 * torch.rand(n, 1, generator=g) - 40)
    sl, sr = torch.rand(n, generator=g) + 0.5, torch.rand(n, generator=g) + 0.5
    V, SL, SR = v.to(device()), sl.to(device()), sr.to(device())
    beta = float(np.float32(1.0 / d))
    rows = np.unique(np.linspace(0, n - 1, 60).astype(int))
    Y = fd.fd_kernel_matmul(x, None, beta, V, sl=SL, sr=SR)
    ref = sl.double().numpy()[rows, None] * ok.kernel_matmul(
        x64[rows], x64, beta, (sr.double()[:, None] * v.double()).numpy())
    assert rel_fro(to_np(Y)[rows], ref) <= TOL_F32
    assert torch.equal(Y, fd.fd_kernel_matmul(x, None, beta, V, sl=SL, sr=SR))
    out = torch.empty_like(Y)
    fd.fd_kernel_matmul_noalloc(x, None, beta, V, out, sl=SL, sr=SR)
    assert torch.equal(Y, out)
    # a NaN reaches every row, an infinity every row whose kernel value is not 0
    for bad in (float("nan"), float("inf")):
        W = V.clone()
        W[n // 2, 0] = bad
        got = to_np(fd.fd_kernel_matmul(x, None, beta, W, sl=SL, sr=SR))
        assert not np.isfinite(got).any()
        assert np.isnan(got).all() == np.isnan(bad)
    assert torch.equal(Y, fd.fd_kernel_matmul(x, None, beta, V, sl=SL, sr=SR))


@pytest.mark.parametrize("n", [513, 5000, 7000])
@pytest.mark.parametrize("kind", ["one point", "decaying", "normal"])
def test_one_column_keeps_small_results(n, kind):
    """Each result by itself: sums far below the column's largest value too.

    The exponent carries a few units of 2^-22 of B = beta log2(e) max|x|^2 < 100
    here (1e-4 of a kernel value); a normal column has results near zero by
    cancellation, so it is compared against its sums without signs.
    """
    case(f"one column n={n} {kind}")
    x, x64 = _points(n, 12, torch.float32)
    g = torch.Generator().manual_seed(5)
    v = torch.randn(n, 1, generator=g)
    if kind == "one point":
        v = torch.zeros(n, 1)
        v[n // 3] = 3.0
    elif kind == "decaying":
        v = torch.exp2(-60 * torch.rand(n, 1, generator=g))
    beta = 4.0
    assert beta * 1.4427 * float(np.square(x64 - x64.mean(0)).sum(1).max()) < 100
    Y = to_np(fd.fd_kernel_matmul(x, None, beta, v.to(device())))
    ref = ok.kernel_matmul(x64, x64, beta, v.double().numpy())
    size = ok.kernel_matmul(x64, x64, beta, v.double().abs().numpy())
    seen = size > 1e-30
    assert seen.sum() > n // 2
    assert (np.abs(Y - ref) <= 1e-4 * size)[seen].all()


@pytest.mark.parametrize("n, span", [(1 << 16, 26.9), (1 << 18, 23.9), (1 << 18, 24.9),
                                     (1 << 18, 25.1), (1 << 20, 22.9), (1 << 20, 23.9)])
def test_one_column_near_the_widest_span(n, span):
    """Two clusters far apart, one with weights 2^span below the other's, in
    sizes where a row's result is little more than its own weight: on both
    sides of the span (2^43 / n) up to which column sums are fixed point.

    Each result to 1e-5 of its sum: 2^-18 of it for the fixed point, and 2e-6
    for the exponents (B = beta log2(e) max|x|^2 < 60).
    """
    case(f"one column n={n} span=2^{span}")
    g = torch.Generator().manual_seed(1)
    x = torch.randn(n, 64, generator=g) * 0.37
    x[::2, 0] += 6.0
    v = torch.ones(n, 1)
    v[1::2] = 2.0 ** -span
    Y = to_np(fd.fd_kernel_matmul(x.to(device()), None, 1.0, v.to(device())))[:, 0]
    rows = 2 * np.linspace(0, n // 2 - 1, 12).astype(int) + 1
    ref = ok.kernel_matmul(x[rows].double().numpy(), x.double().numpy(), 1.0, v.double().numpy())[:, 0]
    assert (np.abs(Y[rows] - ref) <= 1e-5 * ref).all()


@pytest.mark.parametrize("n", [300, 1500, 6500])
def test_one_column_eigensolve_matches_a_wider_one(n):
    """Block width 1 runs its products as single columns (300: in the full space)."""
    case("eigensolve with one column per block")
    x, _ = _points(n, 3, torch.float32)
    a = fd.fd_block_lanczos(x, 0.5, 2, 1)
    b = fd.fd_block_lanczos(x, 0.5, 2, 4)
    assert np.allclose(a.evals[:2], b.evals[:2], rtol=0, atol=1e-6)

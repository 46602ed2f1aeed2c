"""Parity at the full sizes of the larger workloads, on sampled rows.

The noisy 6-torus at n = 262,144 (D = 12, b = 32), the molecule-like set at
N = 2^20 (D = 30, b = 32) and the bfloat16 stress set at N = 2^21 (D = 64,
b = 64), each through the kernels and launch configurations the bench legs
time.  The oracle evaluates the float64 difference-form definition on a
seeded subset of output rows against all N columns: row sums q_S, raw K V,
s on those rows (from the device's q for the other points), the normalised
product diag(s) K diag(s) V with the device's s, and for the molecule set
the true residuals (M phi - theta phi)_S of the top-64 Ritz pairs.

Completeness of the top-64 set at these sizes is pinned on grid tori, whose
spectrum has a closed form at any size (Kronecker product of circulants): the
8^6 grid (262,144 points in R^12, the noisy-6-torus shapes) and the 4^10 grid
(2^20 points in R^20, the D <= 30 layout of the molecule-like set), both with
b = 32 and k = 64.
"""
import numpy as np
import pytest
import torch

from gpu_util import TOL_BF16, TOL_F32, case, device, rel_fro, to_dev, to_np
from oracle import kernel as ok
from oracle import torus_grid as tg
from paper_2609_38198_amd import _lib as fd
from paper_2609_38198_amd import inputs

pytestmark = pytest.mark.gpu

ALPHA = 0.5


def _degree_and_products(X_dev, X64, beta, V, rows, tol):
    dev = device()
    deg = fd.fd_degree(X_dev, beta, ALPHA)
    q = to_np(deg.q)
    s = to_np(deg.s)
    Vd = to_dev(V, dev)
    Y0 = to_np(fd.fd_kernel_matmul(X_dev, None, beta, Vd))
    Y = to_np(fd.fd_kernel_matmul(X_dev, None, beta, Vd, sl=deg.s, sr=deg.s))
    ones = np.ones((X64.shape[0], 1))
    q_ref = ok.kernel_matmul(X64, None, beta, ones, rows=rows, threads=8)[:, 0]
    assert rel_fro(q[rows], q_ref) <= tol
    # s on the sampled rows from w = q^-alpha of every point (device q, checked above on S)
    w = q ** -ALPHA
    t_ref = ok.kernel_matmul(X64, None, beta, w[:, None], rows=rows, threads=8)[:, 0]
    s_ref = w[rows] / np.sqrt(w[rows] * t_ref)
    assert rel_fro(s[rows], s_ref) <= tol
    y0_ref = ok.kernel_matmul(X64, None, beta, V, rows=rows, threads=8)
    assert rel_fro(Y0[rows], y0_ref) <= tol
    y_ref = ok.kernel_matmul(X64, None, beta, V, sl=s, sr=s, rows=rows, threads=8)
    assert rel_fro(Y[rows], y_ref) <= tol
    return deg, s


@pytest.mark.parametrize("beta", [0.5, 8.0])
def test_noisy_torus6_262144(beta):
    w = inputs.torus6_noisy()
    X = w.X.astype(np.float32)
    V = inputs.random_block(w.N, w.b, seed=21)
    rows = np.random.default_rng(22).choice(w.N, 48, replace=False)
    case(f"full size noisy 6-torus N={w.N} D={w.D} b={w.b} beta={beta}")
    _degree_and_products(to_dev(X, device()), X.astype(np.float64), beta, V, rows, TOL_F32)


def test_molecule_2_20_products_and_lanczos_residuals():
    w = inputs.molecule()
    beta = w.betas[0]
    X = w.X.astype(np.float32)
    X64 = X.astype(np.float64)
    V = inputs.random_block(w.N, w.b, seed=23)
    rows = np.random.default_rng(24).choice(w.N, 24, replace=False)
    case(f"full size molecule N={w.N} D={w.D} b={w.b}")
    Xd = to_dev(X, device())
    _, s = _degree_and_products(Xd, X64, beta, V, rows, TOL_F32)
    case(f"full size molecule lanczos k={w.k} b={w.b}")
    e = fd.fd_block_lanczos(Xd, beta, w.k, w.b, alpha=ALPHA, allow_not_converged=True)
    phi = to_np(e.evecs)
    theta = np.asarray(e.evals)
    assert e.info["nconv"] == w.k and abs(theta[0] - 1.0) <= 1e-6
    # (M phi)_S = s_S (K (s phi))_S with the device's s (checked on S above)
    mphi = ok.kernel_matmul(X64, None, beta, phi, sl=s, sr=s, rows=rows, threads=8)
    r = mphi - phi[rows] * theta[None, :]
    # every entry of a residual is at most its norm (<= the solver's 1e-5);
    # the slack covers the float32 operator's own error (~1e-6 relative)
    assert np.abs(r).max() <= 1.5e-5, np.abs(r).max()
    assert np.abs(phi.T @ phi - np.eye(w.k)).max() <= 1e-5


def test_stress_bf16_2_21_product_and_20_iterations():
    # the bfloat16 stress set at its full size: the raw product on 64 sampled
    # rows, then the 20 block iterations of the bench leg (b = 64, basis of 16
    # blocks, 64 kept) and the true residuals (M phi - theta phi)_S of all 64
    # Ritz pairs with the exact operator on 32 sampled rows
    st = inputs.stress()
    beta = st.betas[0]
    X64 = st.X_f64()
    V = inputs.random_block(st.N, st.b, seed=25)
    rows = np.random.default_rng(26).choice(st.N, 64, replace=False)
    case(f"full size bf16 stress N={st.N} D={st.D} b={st.b}")
    Xd = to_dev(st.X, device())
    Y0 = to_np(fd.fd_kernel_matmul(Xd, None, beta, to_dev(V, device())))
    ref = ok.kernel_matmul(X64, None, beta, V, rows=rows, threads=8)
    err = rel_fro(Y0[rows], ref)
    print(f"bf16 full size product rel err {err:.2e}")
    assert err <= TOL_BF16

    case(f"full size bf16 stress: 20 block iterations k=64 b={st.b}")
    o = fd.default_opts(max_matvecs=20, max_basis_blocks=16, keep=64)
    e = fd.fd_block_lanczos(Xd, beta, 64, st.b, alpha=ALPHA, opts=o, allow_not_converged=True)
    assert e.info["block_matvecs"] <= 20
    phi = to_np(e.evecs)
    theta = np.asarray(e.evals)
    deg = fd.fd_degree(Xd, beta, ALPHA)
    q, s = to_np(deg.q), to_np(deg.s)
    rs = rows[:32]
    # s on the sampled rows from the device's q elsewhere (bfloat16 bar)
    ones = np.ones((st.N, 1))
    q_ref = ok.kernel_matmul(X64, None, beta, ones, rows=rs, threads=8)[:, 0]
    assert rel_fro(q[rs], q_ref) <= TOL_BF16
    w = q ** -ALPHA
    t_ref = ok.kernel_matmul(X64, None, beta, w[:, None], rows=rs, threads=8)[:, 0]
    assert rel_fro(s[rs], w[rs] / np.sqrt(w[rs] * t_ref)) <= TOL_BF16
    mphi = ok.kernel_matmul(X64, None, beta, phi, sl=s, sr=s, rows=rs, threads=8)
    lhs = phi[rs] * theta[None, :]
    dev_r = rel_fro(lhs, mphi)
    print(f"bf16 20 iterations: nconv {e.info['nconv']}, solver max residual "
          f"{e.info['max_residual']:.2e}, exact-operator residual on 32 rows "
          f"{dev_r:.2e} (relative), theta0 {theta[0]:.8f}")
    # the Ritz pairs are eigenpairs of the bfloat16 operator to the solver's
    # tolerance; against the exact operator they hold to the bfloat16 product bar
    assert e.info["nconv"] == 64 and e.info["max_residual"] <= 1e-5
    assert dev_r <= TOL_BF16
    assert abs(theta[0] - 1.0) <= TOL_BF16
    assert np.abs(phi.T @ phi - np.eye(64)).max() <= 1e-5


@pytest.mark.parametrize("counts", [(8,) * 6, (4,) * 10])
def test_grid_torus_top64_closed_form(counts):
    # every one of the 64 leading eigenvalues against the closed form: the
    # computed set is the complete top 64 (the cut falls inside a degenerate
    # cluster, where any basis of the eigenspace is a valid answer)
    X = inputs.grid_torus_points(counts).astype(np.float32)
    N, D = X.shape
    beta = 1.0
    ref = tg.operator_eigs(counts, beta)[:64]
    dev = device()
    case(f"lanczos grid torus {counts[0]}^{len(counts)} N={N} D={D} b=32 k=64")
    e = fd.fd_block_lanczos(to_dev(X, dev), beta, 64, 32)
    got = np.asarray(e.evals)
    assert np.all(np.abs(got - ref) <= np.maximum(1e-5 * np.abs(ref), 1e-6)), (
        np.abs(got - ref).max(), e.info)
    assert max(e.residuals) <= 1e-5
    phi = to_np(e.evecs)
    assert np.abs(phi.T @ phi - np.eye(64)).max() <= 1e-5



def test_more_pack_threads_than_one_launch_holds():
    """540 million columns: their packs and that of V take 8 threads a column,
    more than the 2^32 of a launch.  All points coincide but the last one, far
    away, so that results are counts (sums of ones, exact in float32 here)."""
    n = 540_000_001
    case(f"packs in slices nc={n} bf16 b=1")
    dev = device()
    need = fd.fd_workspace_size(fd.FD_OP_KERNEL_MATMUL, 3, n, 1, 1)
    if torch.cuda.mem_get_info()[0] < need + (16 << 30):
        pytest.skip("not enough free device memory")
    xc = torch.zeros(n, 1, dtype=torch.bfloat16, device=dev)
    xc[-1] = 64.0
    xr = torch.tensor([[0.0], [64.0], [32.0]], dtype=torch.bfloat16, device=dev)
    V = torch.ones(n, 1, device=dev)
    V[-1] = 7.0
    ws = torch.empty(need, dtype=torch.uint8, device=dev)
    Y = to_np(fd.fd_kernel_matmul(xr, xc, 1.0, V, ws=ws))[:, 0]
    assert list(Y) == [n - 1, 7.0, 0.0]

"""The dense eigensolve on both sides of the line between its two paths (one
workgroup up to 56 columns, block Jacobi above: four blocks of 16 and more, odd
sizes with a padding block), through eigensolves of the full space.

The eigenvalues are those of the float64 operator to the stated eigenvalue bar
(1e-6 absolute), the vectors orthonormal to 1e-5.
"""
import numpy as np
import pytest
import torch

from gpu_util import case, device, to_np
from oracle import eig as oe
from paper_2609_38198_amd import _lib as fd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 33, 55, 56, 57, 64, 65, 97, 160, 193])
def test_full_space_eigensolve(n):
    case(f"dense eigensolve m={n}")
    x = torch.randn(n, 3, generator=torch.Generator().manual_seed(n))
    k = min(n, 24)
    e = fd.fd_block_lanczos(x.to(device()), 0.3, k, 8)
    ref = oe.spectrum(x.double().numpy(), float(np.float32(0.3)), 0.5, k)
    assert np.abs(np.array(e.evals[:k]) - ref.evals[:k]).max() <= 1e-6
    phi = to_np(e.evecs)
    assert np.abs(phi.T @ phi - np.eye(k)).max() <= 1e-5

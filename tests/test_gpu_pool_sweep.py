"""The pool sweep against the gradient of the ansatz with the operator appended
at angle 0: lists within the entries a wave loads ahead (256) and longer ones,
tiles of few and many gates, real and complex amplitudes.

Tolerance: two orders of the same sums of at most 2^12 products per tile with
coefficients below 100: 2^-52 * 100 * sqrt(4096) = 1.4e-12; 1e-11 allowed.
"""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first)

import paper_2311_01242_amd as vq
from vqe_inputs import random_integrals, uniform_theta

pytestmark = pytest.mark.gpu
TOL = 1e-11


@pytest.mark.parametrize("real", [True, False])
@pytest.mark.parametrize("n,ne", [(6, 3), (12, 6), (17, 8), (20, 10), (21, 6)])
def test_pool_sweep(n, ne, real):
    H = vq.Hamiltonian.from_integrals(n, *random_integrals(n, 4300 + n))
    pool = vq.Ansatz.uccsd(n, ne)
    chosen = np.unique(np.linspace(0, pool.n_params - 1, 5).astype(np.int32))
    theta = uniform_theta(n, chosen.size)
    vq.set_real(real)
    try:
        g = vq.pool_gradient(H, pool.select(chosen), pool, ne, theta)
        g = g[1] if isinstance(g, tuple) else g
        for k in np.unique(np.linspace(0, pool.n_params - 1, 9).astype(np.int32)):
            A = pool.select(np.append(chosen, k).astype(np.int32))
            _, ref = vq.energy_grad(H, A, ne, np.append(theta, 0.0))
            assert abs(g[k] - ref[-1]) < TOL
    finally:
        vq.set_real(True)

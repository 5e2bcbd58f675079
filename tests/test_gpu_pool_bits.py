"""Pool gradients on both sides of the gate count that decides their block bits
(16), against 12 block bits.

Tolerance: as between any two tilings, the order of a sum: 2^-52 * 100 *
sqrt(2000) = 1e-12; 1e-11 allowed.
"""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first)

import paper_2311_01242_amd as vq
from vqe_inputs import random_integrals, uniform_theta

pytestmark = pytest.mark.gpu
TOL = 1e-11


@pytest.mark.parametrize("real", [True, False])
@pytest.mark.parametrize("n,ne", [(18, 9), (20, 10), (21, 8)])
@pytest.mark.parametrize("gates", [1, 15, 16])
def test_pool_block_bits(n, ne, gates, real):
    H = vq.Hamiltonian.from_integrals(n, *random_integrals(n, 5500 + n))
    pool = vq.Ansatz.uccsd(n, ne)
    A = pool.select(np.linspace(0, pool.n_params - 1, gates).astype(np.int32))
    theta = uniform_theta(gates, gates)
    vq.set_real(real)
    try:
        e0, g0 = vq.pool_gradient(H, A, pool, ne, theta)
        vq.set_tuning(n, False, 65536, 65536, 12)
        e1, g1 = vq.pool_gradient(H, A, pool, ne, theta)
    finally:
        vq.set_tuning(n, False)
        vq.set_real(True)
    assert abs(e0 - e1) < TOL and np.abs(g0 - g1).max() < TOL

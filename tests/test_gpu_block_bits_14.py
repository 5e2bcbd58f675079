"""14 block bits for the tiled runs: the plans exist and agree with the chosen
block bits (no refusal is passed over).

Tolerance: as between any two tilings, the order of an energy's or gradient
component's sums: 2^-52 * 100 * sqrt(2000) = 1e-12; 1e-11 allowed.
"""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first)

import paper_2311_01242_amd as vq
from vqe_inputs import random_integrals, uniform_theta

pytestmark = pytest.mark.gpu
TOL = 1e-11


@pytest.mark.parametrize("real", [True, False])
@pytest.mark.parametrize("n,ne", [(17, 8), (18, 9), (20, 6), (20, 12), (22, 5)])
def test_block_bits_14(n, ne, real):
    A = vq.Ansatz.uccsd(n, ne)
    H = vq.Hamiltonian.from_integrals(n, *random_integrals(n, 5100 + n))
    theta = uniform_theta(n, A.n_params)
    vq.set_real(real)
    try:
        e0, g0 = vq.energy_grad(H, A, ne, theta)
        vq.set_tuning(n, False, 65536, 65536, 14)
        e1, g1 = vq.energy_grad(H, A, ne, theta)
    finally:
        vq.set_tuning(n, False)
        vq.set_real(True)
    assert abs(e0 - e1) < TOL and np.abs(g0 - g1).max() < TOL

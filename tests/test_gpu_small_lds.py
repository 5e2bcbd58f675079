"""Small-sector evaluations whose launches take more than 64 KiB of LDS: complex
amplitudes of the largest sector (1,716 strings: 81 KB in the reverse sweep) and
programs of several hundred gates, against the full-vector kernels, alone and in
batches.

Tolerance: as for any small sector, an energy sums at most 200 terms with
coefficients below 100 over normalised amplitudes; the rounding of k gates adds
at most k 2^-52 100 = 2e-11 for 1,000 gates; 5e-11 allowed.
"""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first)

import paper_2311_01242_amd as vq
from vqe_inputs import random_integrals, uniform_theta

pytestmark = pytest.mark.gpu
TOL = 5e-11


@pytest.mark.parametrize("n,k,gates,real", [(13, 6, 0, False), (13, 7, 0, False), (13, 6, 400, True), (13, 6, 1024, True),
                                            (13, 6, 1024, False), (12, 6, 700, True), (6, 3, 1024, False)])
def test_beyond_64_kib(n, k, gates, real):
    H = vq.Hamiltonian.pairs_from_integrals(n, *random_integrals(2 * n, 4300 + n))
    A = vq.Ansatz.puccd(n, k)
    if gates:   # one angle per gate
        A = A.select(np.random.default_rng(gates).integers(0, A.n_params, gates).astype(np.int32))
    theta = uniform_theta(n + k, A.n_params, -0.6, 0.6)
    vq.set_real(real)
    try:
        e0, g0 = vq.energy_grad(H, A, k, theta)
        b = vq.Batch([H] * 3, [A] * 3, [k] * 3)
        eb, gb = b.energy_grad(np.tile(theta, 3))
        assert b.work()[7] == (3.0 if real else 0.0)
        b.close()
        vq.set_packed(False)
        try:
            e1, g1 = vq.energy_grad(H, A, k, theta)
        finally:
            vq.set_packed(True)
    finally:
        vq.set_real(True)
    assert abs(e0 - e1) < TOL and np.abs(g0 - g1).max() < TOL
    assert np.abs(eb - e1).max() < TOL and np.abs(gb.reshape(3, -1) - g1).max() < TOL

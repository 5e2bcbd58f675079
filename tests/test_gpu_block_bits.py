"""The block bits chosen for the tiled runs against 12 and 14 block bits, at
both ends of the rule (18 to 22 qubits, sectors above and below the whole-state
limit), real and complex amplitudes, alone and in batches.

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
@pytest.mark.parametrize("n,ne,count", [(17, 8, 1), (18, 9, 1), (18, 4, 2), (19, 10, 3), (20, 5, 1), (20, 6, 2),
                                        (20, 12, 1), (22, 5, 1), (23, 4, 1)])
def test_block_bits(n, ne, count, real):
    A = vq.Ansatz.uccsd(n, ne)
    Hs = [vq.Hamiltonian.from_integrals(n, *random_integrals(n, 3700 + i)) for i in range(count)]
    th = np.concatenate([uniform_theta(3700 + i, A.n_params) for i in range(count)])

    def run():
        if count == 1:
            return vq.energy_grad(Hs[0], A, ne, th)
        b = vq.Batch(Hs, [A] * count, [ne] * count)
        try:
            return b.energy_grad(th)
        finally:
            b.close()

    vq.set_real(real)
    try:
        e0, g0 = run()
        for L in (12, 14):
            vq.set_tuning(n, count > 1, 65536, 65536, L)
            try:
                e1, g1 = run()
            except vq.VQEError:   # 14 bits: a tile above the run kernels' largest
                assert L == 14
                continue
            finally:
                vq.set_tuning(n, count > 1)
            assert np.abs(e0 - e1).max() < TOL and np.abs(g0 - g1).max() < TOL
    finally:
        vq.set_real(True)

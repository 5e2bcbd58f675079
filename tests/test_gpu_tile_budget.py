"""Full-vector tiles chosen by the program's masks (lone states up to 20 qubits)
against tiles of 512 amplitudes and of 64 KiB: Pauli rotations on few, many and
all qubits, excitations on full vectors, and mixtures of wide and narrow strings.

Tolerance: the same gates in the same order; the sums of an energy or gradient
component over tiles differ in order: 2^-52 * 100 * sqrt(2^16) = 6e-12, 2e-11
allowed.
"""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first)

import paper_2311_01242_amd as vq
from vqe_inputs import random_integrals, uniform_theta

pytestmark = pytest.mark.gpu
TOL = 2e-11


def _program(n, kind):
    rng = np.random.default_rng(n)
    if kind == "uccsd":
        return vq.Ansatz.uccsd(n, n // 2)
    if kind == "bk":
        return vq.Ansatz.uccsd_map(n, n // 2, "bk")
    gates = 150
    x = rng.integers(0, 1 << n, gates).astype(np.uint32)
    if kind == "narrow":
        x &= np.uint32(1) << rng.integers(0, n, gates).astype(np.uint32)
    elif kind == "mixed":
        x[20:] &= rng.integers(0, 1 << n, gates - 20).astype(np.uint32) & rng.integers(0, 1 << n, gates - 20).astype(np.uint32)
    return vq.Ansatz.from_rotations(n, gates, x, rng.integers(0, 1 << n, gates).astype(np.uint32),
                                    np.arange(gates, dtype=np.int32), rng.uniform(0.5, 1.5, gates))


@pytest.mark.parametrize("kind", ["wide", "narrow", "mixed", "uccsd", "bk"])
@pytest.mark.parametrize("n", [2, 9, 10, 11, 12, 13, 16])
def test_tiles(n, kind):
    H = vq.Hamiltonian.from_integrals_map(n, "bk" if kind == "bk" else "jw", *random_integrals(n, 4900 + n))
    A, ne = _program(n, kind), n // 2
    theta = uniform_theta(n, A.n_params)
    vq.set_packed(False)
    try:
        e0, g0 = vq.energy_grad(H, A, ne, theta)
        for amps in (512, 4096):
            vq.set_tuning(n, False, 16 * amps, 32 * min(amps, 2048), min(n, 12))
            e1, g1 = vq.energy_grad(H, A, ne, theta)
            assert abs(e0 - e1) < TOL and np.abs(g0 - g1).max(initial=0.0) < TOL
    finally:
        vq.set_tuning(n, False)
        vq.set_packed(True)

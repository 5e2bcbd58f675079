"""Tiled runs with their pairs divided among 4 to 16 waves (which meet only
where a stretch of gates ends) against runs of a single wave: programs with
long stretches (UCCSD), short ones (k-UpCCGSD), repeated and single gates,
unequal threads in the two passes, tiles of few and many pairs.

Tolerance: the same rotations in the same order; the sums of a gradient
component over waves differ in order: 2^-52 * 100 * sqrt(2000) = 1e-12, 1e-11
allowed.
"""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first)

import paper_2311_01242_amd as vq
from vqe_inputs import random_integrals, uniform_theta

pytestmark = pytest.mark.gpu
TOL = 1e-11


def _ansatz(n, ne, kind):
    if kind.startswith("kup"):
        return vq.Ansatz.kupccgsd(n, ne, int(kind[3:]))
    if kind == "twice":
        return vq.Ansatz.uccsd_trotter(n, ne, 2)
    A = vq.Ansatz.uccsd(n, ne)
    if kind == "last":
        return A.select(np.array([A.n_params - 1], dtype=np.int32))
    if kind == "mixed":   # neighbours with different created orbitals
        return A.select(np.arange(A.n_params, dtype=np.int32)[::7])
    return A


@pytest.mark.parametrize("real", [True, False])
@pytest.mark.parametrize("n,ne,kind", [(12, 6, "uccsd"), (13, 4, "twice"), (18, 9, "uccsd"), (18, 9, "kup1"),
                                       (19, 7, "mixed"), (20, 10, "last"), (21, 10, "uccsd")])
def test_waves(n, ne, kind, real):
    H = vq.Hamiltonian.from_integrals(n, *random_integrals(n, 3900 + n))
    A = _ansatz(n, ne, kind)
    theta = uniform_theta(n, A.n_params)
    vq.set_real(real)
    vq.set_tile_cap(n, False, 2400 if n >= 18 else 300)   # 12 and 13 qubits: tiles, not the whole state
    try:
        vq.set_run_threads(n, False, 64, 64)
        e0, g0 = vq.energy_grad(H, A, ne, theta)
        for threads in ((256, 256), (512, 512), (1024, 1024), (1024, 256)):
            vq.set_run_threads(n, False, *threads)
            e1, g1 = vq.energy_grad(H, A, ne, theta)
            assert abs(e0 - e1) < TOL and np.abs(g0 - g1).max() < TOL
    finally:
        vq.set_run_threads(n, False)
        vq.set_tile_cap(n, False)
        vq.set_real(True)

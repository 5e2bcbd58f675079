"""Whole-state ansatz passes (k_whole.hip: the sector in one workgroup's LDS,
real amplitudes) against the tiled runs and the complex path: gates of no pair
up to many per thread, one and several segments of narrow and wide gates, odd
qubit counts, open shells, a single gate, repeated gates; alone and in batches.

Tolerance: a gate rounds an amplitude (norm 1 state) by about 2^-52, a pass of
at most 1,500 gates an energy or gradient component, with coefficients below
100, by about 2^-52 * 100 * sqrt(1500) = 9e-13; 1e-11 allowed.
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
    return A.select(np.array([A.n_params - 1], dtype=np.int32)) if kind == "last" else A


def _paths(f, n, batched=False):
    """f's results by the whole-state passes, the tiled runs and complex amplitudes."""
    out = [f()]
    vq.set_tile_cap(n, batched, 16)   # below the sector (of more than 16)
    try:
        out.append(f())
    finally:
        vq.set_tile_cap(n, batched, 0)
    vq.set_real(False)
    try:
        out.append(f())
    finally:
        vq.set_real(True)
    return out


@pytest.mark.parametrize("n,ne,kind", [(4, 2, "uccsd"), (5, 2, "last"), (7, 3, "uccsd"), (8, 4, "kup2"), (10, 5, "twice"),
                                       (12, 6, "kup3"), (13, 6, "uccsd"), (14, 5, "uccsd"), (14, 7, "twice"),
                                       (15, 7, "uccsd"), (15, 8, "kup2"), (16, 8, "last"),
                                       (16, 8, "kup1"), (16, 9, "uccsd"), (17, 8, "uccsd")])
def test_whole_state_passes(n, ne, kind):
    H = vq.Hamiltonian.from_integrals(n, *random_integrals(n, 3100 + n))
    A = _ansatz(n, ne, kind)
    theta = uniform_theta(n, A.n_params)
    for grad in (True, False):
        (e0, g0), *rest = _paths(lambda: vq.energy_grad(H, A, ne, theta, grad=grad), n)
        for e1, g1 in rest:
            assert abs(e0 - e1) < TOL
            assert not grad or np.abs(g0 - g1).max() < TOL
    # the same call twice: nothing of the first stays
    e2, g2 = vq.energy_grad(H, A, ne, theta)
    e0, g0 = vq.energy_grad(H, A, ne, theta)
    assert e0 == e2 and np.array_equal(g0, g2)


@pytest.mark.parametrize("n,ne,kind,count", [(6, 3, "uccsd", 9), (12, 6, "kup2", 3), (15, 7, "uccsd", 20)])
def test_whole_state_batches(n, ne, kind, count):
    Hs = [vq.Hamiltonian.from_integrals(n, *random_integrals(n, 3300 + i)) for i in range(count)]
    A = _ansatz(n, ne, kind)
    th = np.concatenate([uniform_theta(3300 + i, A.n_params) for i in range(count)])

    def run():
        b = vq.Batch(Hs, [A] * count, [ne] * count)
        try:
            return b.energy_grad(th)
        finally:
            b.close()

    (e0, g0), *rest = _paths(run, n, batched=True)
    for e1, g1 in rest:
        assert np.abs(e0 - e1).max() < TOL and np.abs(g0 - g1).max() < TOL


def test_more_gates_than_fit():
    """Angles of more gates (7,200) than LDS holds beside the state: tiled
    runs.  The bound above is 2e-12 for them."""
    n, ne = 16, 8
    H = vq.Hamiltonian.from_integrals(n, *random_integrals(n, 3500))
    A = vq.Ansatz.uccsd_trotter(n, ne, 20)
    theta = uniform_theta(35, A.n_params)
    (e0, g0), *rest = _paths(lambda: vq.energy_grad(H, A, ne, theta), n)
    for e1, g1 in rest:
        assert abs(e0 - e1) < TOL and np.abs(g0 - g1).max() < TOL

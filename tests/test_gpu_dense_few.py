"""Full-vector H-apply with few groups (waves take outputs of their own instead of
sharing the groups) and with enough outputs for every workgroup: expectation
values and the gradient of a rotation, against NumPy on the same strings.
Diagonal Hamiltonians of one group in one to three chunks, one to four groups
(around the number of waves), many groups on 20 qubits, dense and sparse states.

Tolerance: energies are sums of at most 600 strings with coefficients below 5
over normalised states: 2^-52 * 600 * 5 * 8 (random signs) = 6e-12, 1e-10 allowed.
"""
import numpy as np
import pytest
import torch

import paper_2311_01242_amd as vq

pytestmark = pytest.mark.gpu
TOL = 1e-10


def _parity(v):
    v = np.asarray(v, np.int64).copy()
    for s in (16, 8, 4, 2, 1):
        v ^= v >> s
    return v & 1


def _strings(n, groups, per, seed):
    """`groups` flip masks (the first one 0) with `per` sign masks each and an even number of Y."""
    rng = np.random.default_rng(seed)
    x = np.repeat(np.concatenate([[0], rng.choice(np.arange(1, 1 << n), groups - 1, replace=False)]), per)
    z = rng.integers(0, 1 << n, x.size)
    odd = _parity(x & z) == 1
    z[odd] ^= (x & -x)[odd]
    return x.astype(np.uint32), z.astype(np.uint32), rng.normal(0.0, 1.0, x.size)


def _apply(x, z, c, psi):
    b = np.arange(psi.size, dtype=np.int64)
    out = np.zeros_like(psi)
    for xk, zk, ck in zip(x, z, c):   # X^x Z^z |b> = (-1)^(b.z) |b ^ x>
        out += ck * ((1 - 2 * _parity(b & int(zk))) * psi)[b ^ int(xk)]
    return out


@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("n,groups,per", [(1, 1, 2), (2, 3, 2), (9, 1, 600), (9, 3, 1), (9, 4, 2), (13, 1, 300), (16, 2, 3),
                                          (17, 1, 40), (17, 4, 1), (18, 3, 5), (20, 1, 12), (20, 6, 2)])
def test_expectation(n, groups, per, sparse):
    x, z, c = _strings(n, groups, per, 10 * n + groups)
    rng = np.random.default_rng(n)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    if sparse:
        psi[rng.random(1 << n) > 0.05] = 0.0
        psi[0] = 1.0
    psi /= np.linalg.norm(psi)
    e = vq.State.wrap(torch.tensor(psi, device="cuda")).expectation(vq.Hamiltonian.from_paulis(n, x, z, c))
    assert abs(e - np.vdot(psi, _apply(x, z, c, psi)).real) < TOL


@pytest.mark.parametrize("n,groups,per", [(1, 1, 2), (5, 2, 3), (12, 1, 300), (16, 3, 2), (18, 5, 2), (20, 1, 4), (20, 5, 1)])
def test_lambda(n, groups, per):
    # one rotation on |ref>: psi = cos|ref> - i sin P|ref>; dE/dtheta = Im <H psi|P psi> with its own strings
    x, z, c = _strings(n, groups, per, 20 * n + groups)
    H = vq.Hamiltonian.from_paulis(n, x, z, c)
    ne, xp, zp, t = n // 2, (1 << n) - 1, 1, 0.7
    A = vq.Ansatz.from_rotations(n, 1, [xp], [zp], [0], [1.0])
    e, g = vq.energy_grad(H, A, ne, np.array([t]))
    eb, gb = vq.Batch([H, H], [A, A], [ne, ne]).energy_grad(np.array([t, t]))
    psi = np.zeros(1 << n, np.complex128)
    psi[(1 << ne) - 1] = 1.0
    b = np.arange(1 << n, dtype=np.int64)
    string = lambda v: 1j * ((1 - 2 * _parity(b & zp)) * v)[b ^ xp]  # noqa: E731
    psi = np.cos(t / 2) * psi - 1j * np.sin(t / 2) * string(psi)
    lam = _apply(x, z, c, psi)
    e_ref, g_ref = np.vdot(psi, lam).real, np.vdot(lam, string(psi)).imag
    assert abs(e - e_ref) < TOL and abs(g[0] - g_ref) < TOL
    assert np.abs(eb - e_ref).max() < TOL and np.abs(gb - g_ref).max() < TOL

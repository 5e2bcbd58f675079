"""Full-vector H-apply and gate runs: expectation values of dense, sparse,
single-amplitude and zero states (only outputs at nonzero amplitudes are
formed), and the gradient of Pauli-rotation programs, against NumPy on the same
strings.  Sizes around the kernels' blocks: one wave of outputs, one or four
outputs per lane (from 17 qubits), one or several Hamiltonian chunks (128
groups, 256 subgroups, 1,024 table entries), whole-state and split rotation
tiles, and 25 qubits (no index list).

Tolerance: energies are sums of at most 400 strings with coefficients below 5
over normalised states: 2^-52 * 400 * 5 * 8 (random signs) = 4e-12, 1e-10 allowed.
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


def _strings(n, k, seed):
    """k folded strings with an even number of Y."""
    rng = np.random.default_rng(seed)
    x, z = rng.integers(0, 1 << n, k), rng.integers(0, 1 << n, k)
    x[: k // 4] = x[k // 4: k // 4 + k // 4]        # groups of several strings
    x[-1] = 0
    odd = _parity(x & z) == 1
    low = x & -x
    z[odd] ^= low[odd]
    return x.astype(np.uint32), z.astype(np.uint32), rng.normal(0.0, 1.0, k)


def _apply(x, z, c, psi):
    b = np.arange(psi.size, dtype=np.int64)
    out = np.zeros_like(psi)
    for xk, zk, ck in zip(x, z, c):   # X^x Z^z |b> = (-1)^(b.z) |b ^ x>
        out += ck * ((1 - 2 * _parity(b & int(zk))) * psi)[b ^ int(xk)]
    return out


def _state(n, kind, seed):
    rng = np.random.default_rng(seed)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    if kind == "sparse":
        psi[rng.random(1 << n) > 0.02] = 0.0
        psi[-1] = 0.3 - 0.1j
    elif kind == "one":
        psi[:] = 0.0
        psi[(1 << n) // 3] = 1j
    elif kind == "zero":
        psi[:] = 0.0
    norm = np.linalg.norm(psi)
    return psi / norm if norm else psi


@pytest.mark.parametrize("kind", ["dense", "sparse", "one", "zero"])
@pytest.mark.parametrize("n,k", [(1, 3), (3, 9), (6, 40), (7, 400), (11, 300), (14, 150), (17, 60), (18, 40)])
def test_expectation(n, k, kind):
    x, z, c = _strings(n, k, 100 * n + k)
    H = vq.Hamiltonian.from_paulis(n, x, z, c)
    psi = _state(n, kind, n)
    t = torch.tensor(psi, device="cuda")
    e = vq.State.wrap(t).expectation(H)
    assert abs(e - np.vdot(psi, _apply(x, z, c, psi)).real) < TOL


def test_expectation_without_index_list():
    n = 25
    x, z = np.array([0, 3, 1 << 24], np.uint32), np.array([1 << 24, 0, 0b100], np.uint32)
    c = np.array([0.7, -0.4, 0.9])
    t = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    rng = np.random.default_rng(4)
    idx = np.unique(rng.integers(0, 1 << n, 300))
    idx = np.unique(np.concatenate([idx, idx ^ 3, idx ^ (1 << 24)]))
    amp = rng.normal(size=idx.size) + 1j * rng.normal(size=idx.size)
    amp /= np.linalg.norm(amp)
    t[torch.tensor(idx, device="cuda")] = torch.tensor(amp, device="cuda")
    at = {int(b): a for b, a in zip(idx, amp)}
    ref = sum(ck * np.conj(at.get(b ^ int(xk), 0.0)) * a * (1 - 2 * int(_parity(b & int(zk))))
              for xk, zk, ck in zip(x, z, c) for b, a in at.items())
    assert abs(vq.State.wrap(t).expectation(vq.Hamiltonian.from_paulis(n, x, z, c)) - ref.real) < TOL


def test_expectation_of_non_finite_state():
    n = 9
    x, z, c = _strings(n, 20, 3)
    t = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    t[5] = complex(float("nan"), 0.0)
    with pytest.raises(vq.VQEError):
        vq.State.wrap(t).expectation(vq.Hamiltonian.from_paulis(n, x, z, c))


@pytest.mark.parametrize("n,gates,k", [(1, 3, 3), (2, 9, 5), (5, 40, 30), (9, 140, 300), (10, 60, 40), (11, 60, 40),
                                       (13, 30, 150), (17, 12, 30)])
def test_rotation_program_gradient(n, gates, k):
    rng = np.random.default_rng(n)
    hx, hz, hc = _strings(n, k, 7 * n)
    H = vq.Hamiltonian.from_paulis(n, hx, hz, hc)
    x, z = rng.integers(0, 1 << n, gates), rng.integers(0, 1 << n, gates)
    x[gates // 3] = 0
    par, sc = rng.integers(0, 3, gates), rng.uniform(-1.5, 1.5, gates)
    theta = rng.uniform(-1, 1, 3)
    ne = n // 2
    A = vq.Ansatz.from_rotations(n, 3, x, z, par, sc)
    b = np.arange(1 << n, dtype=np.int64)

    def string(v, i):   # Hermitian P = i^#Y X^x Z^z
        return 1j ** bin(int(x[i] & z[i])).count("1") * ((1 - 2 * _parity(b & int(z[i]))) * v)[b ^ int(x[i])]

    def rotate(v, i, s):
        a = 0.5 * s * sc[i] * theta[par[i]]
        return np.cos(a) * v - 1j * np.sin(a) * string(v, i)

    psi = np.zeros(1 << n, np.complex128)
    psi[(1 << ne) - 1] = 1.0
    for i in range(gates):
        psi = rotate(psi, i, 1.0)
    lam = _apply(hx, hz, hc, psi)
    e_ref, g_ref = np.vdot(psi, lam).real, np.zeros(3)
    for i in reversed(range(gates)):
        g_ref[par[i]] += sc[i] * np.vdot(lam, string(psi, i)).imag
        psi, lam = rotate(psi, i, -1.0), rotate(lam, i, -1.0)
    e, g = vq.energy_grad(H, A, ne, theta)
    assert abs(e - e_ref) < TOL and np.abs(g - g_ref).max() < TOL
    assert abs(vq.energy_grad(H, A, ne, theta, grad=False)[0] - e_ref) < TOL
    eb, gb = vq.Batch([H, H], [A, A], [ne, ne]).energy_grad(np.concatenate([theta, theta]))
    assert np.abs(eb - e_ref).max() < TOL and np.abs(gb.reshape(2, 3) - g_ref).max() < TOL

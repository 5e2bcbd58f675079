"""Kernels that a call launches, where a rule chooses among several: counted with
the profiler, by names."""
import collections

import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import paper_2311_01242_amd as vq
from vqe_inputs import random_integrals, uniform_theta

pytestmark = pytest.mark.gpu


def launches(call):
    """Launches of the call by kernel name (no template arguments), after a first call."""
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    count = collections.Counter()
    for e in p.key_averages():
        if "vqe::" in e.key:
            count[e.key.split("vqe::")[1].split("<")[0].split("(")[0]] += e.count
    assert count
    return count


@pytest.mark.parametrize("n,listed", [(2, False), (4, False), (10, False), (16, True)])
def test_expectation_lists_nonzero_amplitudes(n, listed):
    H = vq.Hamiltonian.from_integrals(n, *random_integrals(n, 4700 + n))
    t = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    t[(1 << (n // 2)) - 1] = 1.0
    s = vq.State.wrap(t)
    got = launches(lambda: s.expectation(H))
    assert got["k_hx_dense"] == 1 and got["k_nz_count"] == int(listed) and sum(got.values()) == (5 if listed else 2)


@pytest.mark.parametrize("n,k", [(16, 1), (18, 20), (20, 3)])
def test_few_strings_need_no_list(n, k):
    rng = np.random.default_rng(n)
    H = vq.Hamiltonian.from_paulis(n, rng.integers(0, 1 << n, k), np.zeros(k, np.uint32), rng.normal(size=k))
    t = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    t[5] = 1.0
    s = vq.State.wrap(t)
    got = launches(lambda: s.expectation(H))
    assert got["k_hx_dense"] == 1 and sum(got.values()) == 2


def _rotations(n, gates, width, seed):
    """Strings on `width` qubits (0: one to four), one angle each."""
    rng = np.random.default_rng(seed)
    x, z = np.zeros(gates, np.uint32), np.zeros(gates, np.uint32)
    for i in range(gates):
        for q in rng.choice(n, min(n, width or int(rng.choice([1, 2, 2, 2, 4]))), replace=False):
            letter = int(rng.integers(1, 4))
            x[i] |= np.uint32((letter & 1) << int(q))
            z[i] |= np.uint32((letter >> 1) << int(q))
    return vq.Ansatz.from_rotations(n, gates, x, z, np.arange(gates, dtype=np.int32), rng.uniform(0.5, 1.5, gates))


@pytest.mark.parametrize("n,width,least,most", [(9, 9, 1, 4), (10, 10, 1, 8), (11, 6, 1, 8), (11, 9, 1, 8), (11, 11, 1, 8),
                                                (14, 0, 16, 100), (16, 0, 16, 100)])
def test_rotation_runs_follow_the_masks(n, width, least, most):
    # wide strings: the tile is the whole state (400 gates in runs of up to 128); narrow ones: small tiles
    H = vq.Hamiltonian.from_paulis(n, [0, 1], [1, 0], [1.0, 0.5])
    A = _rotations(n, 400, width, n)
    theta = uniform_theta(n, 400)
    got = launches(lambda: vq.energy_grad(H, A, n // 2, theta))
    assert least <= got["k_rot_fwd"] + got["k_pauli"] <= most
    assert least <= got["k_rot_adj"] + got["k_adj_pauli"] <= most


@pytest.mark.parametrize("n,ne,kind,tiled", [(16, 8, "uccsd", False), (17, 8, "uccsd", True), (17, 8, "kup", True),
                                             (17, 9, "kup", True), (17, 7, "kup", False), (17, 8, "few", False),
                                             (22, 5, "uccsd", False)])
def test_lone_states_in_large_sectors_take_tiles(n, ne, kind, tiled):
    H = vq.Hamiltonian.from_integrals(n, *random_integrals(n, 4800 + n))
    A = vq.Ansatz.kupccgsd(n, ne, 2) if kind == "kup" else vq.Ansatz.uccsd(n, ne)
    if kind == "few":
        A = A.select(np.arange(0, A.n_params, 30, dtype=np.int32))
    theta = uniform_theta(n, A.n_params)
    value = []
    got = launches(lambda: value.append(vq.energy_grad(H, A, ne, theta)))
    assert (got["k_prun"] > 0) == tiled and got["k_whole_fwd"] == got["k_whole_adj"] == int(not tiled)
    # a batch member of the same kind: whole states; sums in another order (2^-52 * 100 * sqrt(9075) = 2e-12)
    b = vq.Batch([H] * 2, [A] * 2, [ne] * 2)
    eb, gb = b.energy_grad(np.tile(theta, 2))
    b.close()
    assert np.abs(eb - value[0][0]).max() < 1e-11 and np.abs(gb.reshape(2, -1) - value[0][1]).max() < 1e-11


def _near_two_body(n, kind):
    """A Hamiltonian near one of two-body integrals: that one (plain), or one without a matrix form."""
    x, z, c = vq.Hamiltonian.from_integrals(n, *random_integrals(n, 77)).terms()
    keep = np.ones(x.size, bool)
    pairs = [k for k in range(x.size) if bin(int(x[k]) & 0xAAAAAAAA).count("1") == 2 and
             bin(int(x[k]) & 0x55555555).count("1") == 2]
    xa, xb = int(x[pairs[0]]) & 0x55555555, int(x[pairs[0]]) & 0xAAAAAAAA
    if kind in ("direction", "constant"):   # a double excitation whose coefficient depends on the hops' directions,
        x = np.append(x, x[pairs[0]])       # with "constant" by little beside a constant that dwarfs all others
        z = np.append(z, z[pairs[0]] ^ np.uint32(xa & -xa) ^ np.uint32(xb & -xb))
        c = np.append(c, 0.3 if kind == "direction" else 1e-5)
        keep = np.ones(x.size, bool)
        if kind == "constant":
            c[(x == 0) & (z == 0)] += 1e10
    elif kind == "chain":        # a sign mask that is no Jordan-Wigner chain
        free = ~(int(x[pairs[0]])) & ((1 << n) - 1)
        z[x == x[pairs[0]]] ^= np.uint32(free & -free)
    elif kind == "diagonal":     # a three-orbital Z string
        x, z, c = np.append(x, np.uint32(0)), np.append(z, np.uint32(0b10110)), np.append(c, 0.37)
        keep = np.ones(x.size, bool)
    return vq.Hamiltonian.from_paulis(n, x[keep], z[keep], c[keep])


@pytest.mark.parametrize("kind", ["plain", "direction", "constant", "chain", "diagonal"])
@pytest.mark.parametrize("n,ne", [(12, 6), (15, 6), (18, 9)])
def test_hamiltonians_without_matrix_form_are_walked(n, ne, kind):
    # 2^-52 * 100 * sqrt(2000) = 1e-12 as for any two forms of the H-apply, 1e-11 allowed; with the
    # constant a gradient component sums products of amplitudes with rounding errors of 2^-53 1e10 = 1e-6
    tol = 1e-5 if kind == "constant" else 1e-11
    H = _near_two_body(n, kind)
    A = vq.Ansatz.uccsd(n, ne)
    theta = uniform_theta(5, A.n_params, -0.3, 0.3)
    value = []
    got = launches(lambda: value.append(vq.energy_grad(H, A, ne, theta)))
    assert (got["k_hx_cross"] > 0) == (kind == "plain") and (got["k_hx_ci"] > 0) == (kind != "plain")
    vq.set_packed(False)
    try:
        e, g = vq.energy_grad(H, A, ne, theta)
    finally:
        vq.set_packed(True)
    assert abs(value[0][0] - e) < max(tol, 1e-15 * abs(e) * 100) and np.abs(value[0][1] - g).max() < tol


@pytest.mark.parametrize("n", [12, 13, 14, 16, 17, 19, 20, 22, 23, 24])
def test_two_body_hamiltonians_have_the_matrix_form(n):
    A = vq.Ansatz.uccsd(n, n // 2).select(np.arange(2, dtype=np.int32))
    for seed in range(3):
        h0, h, g = random_integrals(n, 5300 + seed)
        H = vq.Hamiltonian.from_integrals(n, h0 + 1e3, 10.0 ** (seed - 1) * h, g)
        got = launches(lambda: vq.energy_grad(H, A, n // 2, np.array([0.1, -0.2])))
        assert got["k_hx_cross"] > 0 and got["k_hx_ci"] == 0


@pytest.mark.parametrize("n", [16, 20, 24])
@pytest.mark.parametrize("kind", ["z", "hubbard", "one-body"])
def test_sparse_hamiltonians_are_walked(n, kind):
    ns = (n + 1) // 2
    chain, g = -(np.eye(ns, k=1) + np.eye(ns, k=-1)), np.zeros((ns,) * 4)
    if kind == "hubbard":
        for i in range(ns):
            g[i, i, i, i] = 4.0
    if kind == "z":
        H = vq.Hamiltonian.from_paulis(n, [0], [1], [1.0])
    else:
        H = vq.Hamiltonian.from_integrals(n, 0.0, chain if kind == "hubbard" else random_integrals(n, 1)[1], g)
    A = vq.Ansatz.uccsd(n, n // 2).select(np.arange(2, dtype=np.int32))
    got = launches(lambda: vq.energy_grad(H, A, n // 2, np.array([0.1, -0.2])))
    assert got["k_hx_cross"] == 0 and got["k_hx_ci"] == 1

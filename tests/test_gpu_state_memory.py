"""Expectation value of a 24-qubit state on a nearly full device: the index list
of its nonzero amplitudes (64 MiB) is left out where it has no room.

Tolerance: three strings of one state against their closed values: 1e-12.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2311_01242_amd as vq

pytestmark = pytest.mark.gpu


def test_expectation_on_a_full_device():
    n = 24
    x, z = np.array([0, 0, 1 << 20], np.uint32), np.array([1, 1 << 23, 0], np.uint32)
    H = vq.Hamiltonian.from_paulis(n, x, z, np.array([0.5, 0.25, 2.0]))
    t = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    t[1] = 0.6
    t[1 ^ (1 << 20)] = 0.8
    stream = torch.cuda.Stream()   # a stream without scratch so far
    torch.cuda.synchronize()
    want = -0.5 + 0.25 + 2.0 * 2 * 0.6 * 0.8
    hold = []
    torch.cuda.empty_cache()
    for _ in range(4):
        free = torch.cuda.mem_get_info()[0]
        if free > 100 << 20:
            hold.append(torch.empty(free - (90 << 20), dtype=torch.uint8, device="cuda"))
    try:
        left = torch.cuda.mem_get_info()[0]
        e = vq.State.wrap(t, stream=C.c_void_p(stream.cuda_stream)).expectation(H)
        after = torch.cuda.mem_get_info()[0]
    finally:
        hold.clear()
        torch.cuda.empty_cache()
    assert left < 128 << 20 and left - after < 48 << 20
    assert abs(e - want) < 1e-12

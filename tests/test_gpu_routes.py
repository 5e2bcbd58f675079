"""Kernels that a call launches, where a rule chooses among several: counted with
the profiler, by names."""
import collections

import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import paper_2311_01242_amd as vq
from vqe_inputs import random_integrals

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

"""Measured HBM traffic is tied to every kernel source whose bytes it counts (CPU)."""
import os
import shutil
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_2311_01242_amd import profiling  # noqa: E402

KERNELS = {"k_prun": "k_packed.hip", "k_whole_fwd": "k_whole.hip", "k_whole_adj": "k_whole.hip", "k_hx_same": "k_hx_mm.hip",
           "k_hx_cross": "k_hx_mm.hip", "k_hx_ci": "k_hx_ci.hip", "k_ci_scatter": "k_hx_ci.hip",
           "k_ci_gather": "k_hx_ci.hip"}


@pytest.mark.parametrize("kernel,source", sorted(KERNELS.items()))
def test_counted_kernels_are_hashed(kernel, source):
    assert kernel + "(" in open(os.path.join(profiling.CSRC, source)).read()
    for name in ([kernel + "<1, 256>", kernel + "<2, 256>"] if kernel == "k_prun" else [kernel]):
        phase = profiling.phase_of("void vqe::" + name)
        assert source in profiling.PHASE_SOURCE[phase] and source in bench.PHASE_KERNELS[phase][1]


@pytest.mark.parametrize("phase", ["forward", "h_apply", "adjoint"])
def test_an_edit_of_any_source_changes_the_hash(phase, tmp_path, monkeypatch):
    sources = profiling.PHASE_SOURCE[phase]
    assert tuple(bench.PHASE_KERNELS[phase][1]) == tuple(sources)
    for s in sources:
        shutil.copy(os.path.join(profiling.CSRC, s), tmp_path / s)
    monkeypatch.setattr(profiling, "CSRC", str(tmp_path))
    monkeypatch.setattr(bench, "CSRC", str(tmp_path))
    first = profiling._sha(sources)
    assert bench.source_hash(sources) == first
    for s in sources:
        (tmp_path / s).write_text((tmp_path / s).read_text() + "\n")
        now = profiling._sha(sources)
        assert now != first and bench.source_hash(sources) == now
        first = now

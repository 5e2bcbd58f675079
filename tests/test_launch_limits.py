"""Grids of batched launches on the CPU: HIP takes less than 2^32 threads in a
grid's x dimension, which a large batch of the matrix-form H-apply (one workgroup
of up to 1,024 threads per row of every state) could exceed.
"""
import os
import shutil
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_01242_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "run_layout.h"
int main() {
    int bad = 0;
    for (int64_t rows : {1, 6, 20, 70, 252, 462, 924, 1716})
        for (int64_t threads : {256, 512, 1024}) {
            const int64_t n = vqe::states_per_launch(rows * threads);
            const bool ok = n >= 8 && n % 8 == 0 && n * rows * threads < (int64_t(1) << 32) &&
                            (n + 8) * rows * threads >= (int64_t(1) << 32);
            if (!ok) std::printf("rows %ld threads %ld: %ld\n", long(rows), long(threads), long(n));
            bad += !ok;
        }
    return bad != 0;
}
"""


def test_states_per_launch(tmp_path):
    cxx = os.environ.get("CXX_HOST", shutil.which("g++") or "g++")
    src, exe = tmp_path / "limits.cpp", tmp_path / "limits"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout

"""LDS of the tiled runs on the CPU: every access of a pass to its gates'
parameters and wave totals lies within the LDS that the launch asks for.

A forward pass stages gate j at entries 2 j and 2 j + 1 (16 bytes each) and
reads entry 2 (j + 1) during gate j; the reverse sweep reads entry 2 (j - 1),
down to -2, and stores `waves` totals of 8 bytes per gate.
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
    int bad = 0, seen = 0;
    for (int vectors : {1, 2})
        for (int vbytes : {8, 16})
            for (int entries : {1, 2, 3, 64, 1599, 2400, 4095, 4096})
                for (int gates : {1, 2, 7, 8, 9, 64, 127, 128})
                    for (int waves : {1, 4, 8, 16}) {
                        const vqe::RunLds l = vqe::tiled_run_lds(vectors, vbytes, entries, gates, waves);
                        const long tile = long(vectors) * (entries + 2) * vbytes;
                        const long low = vectors == 1 ? 0 : -2, high = vectors == 1 ? 2 * gates : 2 * gates - 1;
                        const bool ok = l.par % 16 == 0 && l.wsum % 16 == 0 && tile <= long(l.par) &&
                                        long(l.par) + 16 * low >= 0 &&
                                        l.par + 16 * size_t(high + 1) <= l.total &&
                                        l.par + 32 * size_t(gates) <= l.wsum &&
                                        (vectors == 1 || l.wsum + 8 * size_t(gates) * waves <= l.total) &&
                                        l.total <= (160u << 10);
                        ++seen;
                        if (!ok && bad++ == 0)
                            std::printf("vectors %d vbytes %d entries %d gates %d waves %d\n", vectors, vbytes, entries,
                                        gates, waves);
                    }
    std::printf("%d of %d\n", bad, seen);
    return bad != 0;
}
"""


def test_parameter_reads_stay_in_lds(tmp_path):
    cxx = os.environ.get("CXX_HOST", shutil.which("g++") or "g++")
    src, exe = tmp_path / "layout.cpp", tmp_path / "layout"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout

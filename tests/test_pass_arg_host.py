"""The fourth argument of a generated pass kernel (single tiles or whole rows
with an expectation epilogue, else the XCD remap) follows the kernel's kind,
also where a row has one tile; the launcher takes it from there. The header is
compiled on the host."""
import os
import subprocess

import pytest

from paper_2609_23664_amd import build

PROGRAM = """
#include "qw_jit.h"
#include <cstdio>
int main() {
    for (int epi = 0; epi < 2; ++epi)
        for (int rows = 1; rows <= 4; rows *= 4)
            for (int remap = 0; remap < 2; ++remap)
                for (int by_tile = 0; by_tile < 2; ++by_tile) {
                    qw::JitKernel k;
                    k.epi = epi != 0;
                    k.row_tiles = rows;
                    std::printf("%d %d %d %d\\n", epi, remap, by_tile, qw::pass_mode_arg(k, remap, by_tile != 0));
                }
}
"""


def test_mode_argument_follows_the_kernel(tmp_path):
    src, exe = tmp_path / "arg.cpp", tmp_path / "arg"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                    build.INCLUDE, "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")[:-1]
    assert len(lines) == 16
    for line in lines:
        epi, remap, by_tile, arg = map(int, line.split())
        assert arg == (by_tile if epi else remap), line


@pytest.mark.parametrize("text", ["remap = pass_mode_arg(k, remap, by_tile);", "k->epi = ks[i].pass && ks[i].epi;"])
def test_launcher_uses_it(text):
    assert text in open(os.path.join(build.CSRC, "qw_jit.cpp")).read()

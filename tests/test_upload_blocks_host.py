"""Workgroups of a plan upload: at most 16 KiB each (one 16-byte read a thread)
until the limit of 64 is reached. The header is compiled on the host."""
import subprocess

from paper_2609_23664_amd import build

PROGRAM = """
#include "qw_kernels.h"
#include <cstdio>
int main() {
    for (unsigned long long k : {1ull, 16384ull, 16385ull, 20480ull, 32752ull, 32768ull, 32769ull, 1048560ull,
                                 1048576ull, 1048577ull, 26214400ull})
        std::printf("%llu %u\\n", k, qw::upload_blocks(k));
}
"""


def test_upload_blocks(tmp_path):
    src, exe = tmp_path / "blocks.cpp", tmp_path / "blocks"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                    build.INCLUDE, "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")[:-1]
    assert len(lines) == 11
    for line in lines:
        size, blocks = map(int, line.split())
        assert blocks == max(1, min(64, -(-size // 16384))), line

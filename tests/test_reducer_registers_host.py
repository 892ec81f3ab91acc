"""Generated reducers keep within a thread's registers: the kernels of 50 terms
on 14 qubits (one tile), on 20 (rows or single tiles) and on 24 (rows) are
compiled as they are at run time and use no scratch memory."""
import re
import subprocess

import numpy as np
import pytest

from paper_2609_23664_amd import binding as B
from paper_2609_23664_amd import build
from workloads import gen


@pytest.mark.parametrize("n,terms", [(14, [50]), (16, [10, 40]), (20, [15, 35]), (24, [5, 9, 10, 26])])
def test_no_scratch(tmp_path, monkeypatch, n, terms):
    monkeypatch.setenv("QW_JIT_CACHE", str(tmp_path / "jit"))
    dump = tmp_path / "dump"
    dump.mkdir()
    monkeypatch.setenv("QW_JIT_DUMP", str(dump))
    B.jit_precompile_terms(n, gen.random_pauli_terms(np.random.default_rng(1000 * n + 50), n, 50))
    texts = [f.read_text() for f in dump.glob("*.hip")]
    assert sorted(int(re.search(r"\bNT = (\d+);", t).group(1)) for t in texts) == terms
    for i, t in enumerate(texts):
        src, asm = tmp_path / f"k{i}.hip", tmp_path / f"k{i}.s"
        src.write_text("#include <hip/hip_runtime.h>\n" + t)
        subprocess.run([build.HIPCC, "-x", "hip", *build.DEVICE, "-O3", "-std=c++17", "-ffp-contract=off", "-I",
                        build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True,
                       capture_output=True)
        assert re.findall(r"; ScratchSize: (\d+)", asm.read_text()) == ["0"]

"""Memory ordering of the generated persistent kernels, read from their text:
the wait between the release fence and the completion counter's add (the
compiler drops the fence's own wait behind the cache write-back, so a counter
could be seen before the states it stands for), and the one behind the acquire
fence before the other waves start."""
from paper_2609_23664_amd import binding as B
from workloads import gen


def test_persistent_kernel_waits_for_its_fences(tmp_path, monkeypatch):
    monkeypatch.setenv("QW_JIT_CACHE", str(tmp_path / "jit"))
    dump = tmp_path / "dump"
    dump.mkdir()
    monkeypatch.setenv("QW_JIT_DUMP", str(dump))
    w = gen.small_vqe(15, 1, 2, 2, 3, seed=9)
    B.jit_precompile_suffix(15, w.suffixes[0], w.terms)
    texts = [t for t in (f.read_text() for f in dump.glob("*.hip")) if "void qw_persist(" in t]
    assert texts
    for t in texts:
        release = t.index('__builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent")')
        add = t.index("__hip_atomic_fetch_add(&sync[kSyncCounters", release)
        assert "__builtin_amdgcn_s_waitcnt(0);" in t[release:add]
        acquire = t.index('__builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent")')
        assert "__builtin_amdgcn_s_waitcnt(0);" in t[acquire:t.index("s_claim = c;", acquire)]

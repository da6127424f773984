"""CPU checks of the kernels' sources: a handover between the lanes of a wave
goes through wave_sync(), whose fences order the lanes' LDS accesses."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def sources():
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_1404_0743_amd", "csrc", "*"))):
        if path.endswith((".hip", ".h", ".cpp")):
            with open(path) as f:
                yield os.path.basename(path), re.sub(r"//[^\n]*", "", f.read())


def test_wave_barrier_stands_between_fences():
    """__builtin_amdgcn_wave_barrier() by itself orders no memory: every one of
    them has a release fence before it and an acquire fence after it."""
    fenced = re.compile(r'__builtin_amdgcn_fence\(__ATOMIC_RELEASE, "wavefront"\);\s*'
                        r'__builtin_amdgcn_wave_barrier\(\);\s*'
                        r'__builtin_amdgcn_fence\(__ATOMIC_ACQUIRE, "wavefront"\);')
    found = 0
    for name, text in sources():
        found += len(fenced.findall(text))
        assert "__builtin_amdgcn_wave_barrier" not in fenced.sub("", text), name
    assert found >= 1

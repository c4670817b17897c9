"""CPU checks of rules that the HIP sources keep and no run shows: they read the sources only."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_17320_amd", "csrc")


def sources():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        with open(path) as f:
            yield os.path.basename(path), re.sub(r"//[^\n]*", "", f.read())


def test_workgroups_of_a_launch_hand_each_other_nothing():
    """Results pass from workgroup to workgroup at launch boundaries only: no counters, flags or fences in device
    memory whose order would have to be argued."""
    for name, text in sources():
        assert not re.findall(r"__hip_atomic_\w+|__threadfence\w*|MEMORY_SCOPE_\w+|__builtin_amdgcn_fence", text), name


def test_assembly_leaves_m0_to_the_compiler():
    """The asynchronous copies get their LDS base as an m0 operand; no asm statement writes m0 behind the compiler's
    back (which merges and moves its own writes of it)."""
    copies = 0
    for name, text in sources():
        for stmt in re.findall(r"\basm\b[^;]*?\((.*?)\)\s*;", text, re.S):
            assert not re.search(r"\bs_\w+\s+m0\b", stmt), (name, stmt)
            if "load_lds" in stmt:
                copies += 1
                assert '"{m0}"' in stmt, (name, stmt)
    assert copies

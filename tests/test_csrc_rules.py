"""CPU checks of rules that the HIP sources keep and no run shows: they read the sources only."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_17320_amd", "csrc")


def sources():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        with open(path) as f:
            yield os.path.basename(path), re.sub(r"//[^\n]*", "", f.read())


# the atomics there are: counters in LDS (the selects' histograms and candidate lists, whose memory all comes from `hist`)
LDS_COUNTERS = {("select.hip", "&h["), ("select.hip", "&list[")}


def handed_over(name, text):
    """What in a source could pass a result from workgroup to workgroup: atomics on anything but the counters in LDS,
    scoped atomics, fences, and reads or writes past the caches that only such a hand-over needs."""
    found = re.findall(r"__(?:hip|scoped|opencl)_atomic_\w+|__atomic_\w+|__sync_\w+|__threadfence\w*|MEMORY_SCOPE_\w+"
                       r"|__builtin_amdgcn_(?:fence|(?:global|flat|ds|raw\w*_buffer|struct\w*_buffer)_atomic)\w*"
                       r"|\b(?:global|flat|buffer)_atomic_\w+|\bvolatile\s+(?!\()(?!\")\w+", text)
    for call, operand in re.findall(r"\b(atomic[A-Z]\w*)\s*\(\s*(&?\s*\w+\s*\[?)", text):
        if (name, operand.replace(" ", "")) not in LDS_COUNTERS:
            found.append(f"{call}({operand}")
    return found


def test_workgroups_of_a_launch_hand_each_other_nothing():
    """Results pass from workgroup to workgroup at launch boundaries only: no counters, flags or fences in device
    memory whose order would have to be argued."""
    for name, text in sources():
        assert not handed_over(name, text), (name, handed_over(name, text))
        if name == "select.hip":                     # ... and `hist` is LDS
            for line in ("int *h = hist + at * NR * 256, *hn = hist + next * NR * 256;", "int *list = hist;", "list = hn;",
                         "extern __shared__ __align__(16) uint32_t score_lds[];", "int *hist = reinterpret_cast<int *>(score_lds);",
                         "__shared__ __align__(16) int hist[3 * 256];"):
                assert text.count(line) == 1, line
            assert len(re.findall(r"\b(?:hist|h|list) =", text)) == 4


def test_the_rule_sees_a_hand_over():
    for planted in ("if (atomicAdd(done, 1) == last) reduce();", "atomicMax(&best[b], v);", "atomicCAS (flag, 0, 1);",
                    "__hip_atomic_fetch_add(p, 1, x, y);", "__atomic_load_n(p, 2);", "volatile int *flag = f;",
                    "__builtin_amdgcn_global_atomic_fadd_f32(p, v);", "global_atomic_add_u32 v0"):
        assert handed_over("kernel.hip", planted), planted
    assert handed_over("kernel.hip", "atomicAdd(&h[i], 1);") and not handed_over("select.hip", "atomicAdd(&h[i], 1);")


def replaced_pointers(text):
    """Operands in scalar registers that an asm statement reads and replaces and that the source does not declare as whole numbers."""
    def number(op):
        return re.search(rf"\b(?:int|unsigned|uint64_t)\b[^;{{}}*]*?\b{op}\b", text) and not re.search(rf"\*(?:const |__restrict__ )?{op}\b", text)
    return [op for stmt in re.findall(r"\basm\b[^;]*?\((.*?)\)\s*;", text, re.S) for op in re.findall(r'"\+s"\s*\((\w+)', stmt) if not number(op)]


def test_assembly_replaces_no_pointers():
    """A pointer that comes out of an asm statement is one of unknown memory to the compiler, and what goes through it are flat accesses, which count as
    LDS operations too: addresses pass as numbers, and arguments that are wanted early are read only."""
    for name, text in sources():
        assert not replaced_pointers(text), (name, replaced_pointers(text))
    assert replaced_pointers('void now(ARG &a) { asm volatile("" : "+s"(a)); }') == ["a"]
    assert replaced_pointers('int n, float *__restrict__ score) { asm volatile("" : "+s"(score), "+s"(n)); }') == ["score"]


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

"""What the prompt kernels' hand-written waits have to say, read from the source: a missing one is a race that need not show."""
import os
import re

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_08856_amd", "csrc", "prefill.hip")


def statements():
    text = re.sub(r"//[^\n]*", "", open(SOURCE).read())
    return [s.strip() for s in text.split(";")]


def test_loads_to_lds_declare_the_register_they_write():
    loads = [s for s in statements() if "global_load_lds" in s]
    assert loads
    for s in loads:
        assert "s_mov_b32 m0" in s and re.search(r':\s*"memory",\s*"m0"\)$', s), s


def test_a_raw_barrier_waits_for_the_loads_and_for_the_wave_s_own_lds_reads():
    """The barrier hands a buffer that this wave has read to the loads of another wave: its reads have to be complete."""
    code = statements()
    at = [i for i, s in enumerate(code) if "__builtin_amdgcn_s_barrier" in s]
    assert len(at) == 2
    for i in at:
        assert re.search(r'asm volatile\("s_waitcnt vmcnt\(%0\) lgkmcnt\(0\)"', code[i - 1]), code[i - 1]

"""Static check of this library's generated gfx950 code: loads that are meant to be in flight together are."""
import os
import re

from test_isa_hazards import CSRC, assemble


def functions(lines):
    """{mangled name: its instructions} of the kernels in an assembly listing."""
    found, name = {}, None
    for line in lines:
        text = line.split(";")[0].strip()
        m = re.match(r"(_Z\w+):$", text)
        if m:
            name = m.group(1)
            found[name] = []
        elif text.startswith(".Lfunc_end"):
            name = None
        elif name and text and not text.startswith("."):
            found[name].append(text)
    return found


def waits_behind_a_load(code):
    return [b for a, b in zip(code, code[1:]) if a.startswith("global_load") and b.startswith("s_waitcnt") and "vmcnt(0)" in b]


def test_the_gathered_filters_of_the_chunk_parallel_forward_do_not_wait_for_each_other(tmp_path):
    """A wave gathers its Toeplitz operands with one load per four taps; a wait behind each made calls with 65 taps up to
    21% slower."""
    kernels = {n: c for n, c in functions(assemble(os.path.join(CSRC, "cp4_kernels.hip"), tmp_path)).items() if "cp4" in n}
    assert len(kernels) >= 8
    for name, code in kernels.items():
        assert not waits_behind_a_load(code), name

"""The kernel for small products: rows that need no words carry nothing of the way of those that do, and the group that K ends in is
asked for as a whole beside them.  Seen in the code built."""
import os
import re
import subprocess

import pytest

import paper_2003_06324_amd as g
from paper_2003_06324_amd import build
from test_wide_store_data import _code_objects


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    """{(type, A K-contiguous, B K-contiguous, A by words, B by words): instructions}"""
    g.load_library()   # (builds it if it is not there)
    objdump = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "llvm", "bin", "llvm-objdump")
    path, found = str(tmp_path_factory.mktemp("code") / "a.co"), {}
    for image in _code_objects(build.LIB):
        if b"gemm_small_kernel" not in image:
            continue
        with open(path, "wb") as f:
            f.write(image)
        kernel = None
        for line in subprocess.run([objdump, "-d", "--no-show-raw-insn", "--demangle", path], check=True, stdout=subprocess.PIPE,
                                   universal_newlines=True).stdout.splitlines():
            m = re.match(r"[0-9a-f]+ <(.*)>:$", line)
            if m:
                m = re.search(r"gemm_small_kernel<([^>]*)>", m.group(1))
                args = m.group(1).split(", ") if m else None
                kernel = found.setdefault((args[0],) + tuple(a == "true" for a in args[1:]), []) if m else None
            elif kernel is not None and line.split("//")[0].strip():
                kernel.append(line.split("//")[0].strip())
    return found


def _longest_run_of_loads(code):
    longest = run = 0
    for line in code:
        if "s_waitcnt" in line and "vmcnt" in line:
            run = 0
        run += line.startswith("global_load")
        longest = max(longest, run)
    return longest


def test_rows_on_words_carry_no_other_way(forms):
    # (427, 707 and 700 instructions; 876, 897 and 909 with the choice made at run time)
    most = {(True, True): 460, (False, True): 740, (True, False): 740}
    for f, code in forms.items():
        if f[0] != "float" and not any(f[3:5]) and any(f[1:3]):
            assert len([c for c in code if not c.startswith(("s_nop", "s_code_end"))]) <= most[f[1:3]], f


def test_the_group_that_k_ends_in_is_requested_as_a_whole(forms):
    by_words = [f for f in forms if any(f[3:5])]
    assert len(by_words) == 2 * 5   # binary16 and bfloat16; one operand or both, the other one K-contiguous or not
    for f in by_words:
        assert _longest_run_of_loads(forms[f]) >= 16, f

"""The kernel for small products: rows that need no words carry nothing of the way of those that do, and the group that K ends in is
asked for as a whole beside them.  Seen in the code built."""
import pytest

from code_util import kernels


@pytest.fixture(scope="module")
def forms():
    """{(type, A K-contiguous, B K-contiguous, A by words, B by words): instructions}"""
    return kernels("gemm_small_kernel")


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
            assert len(code) <= most[f[1:3]], f


def test_the_group_that_k_ends_in_is_requested_as_a_whole(forms):
    by_words = [f for f in forms if any(f[3:5])]
    assert len(by_words) == 2 * 5   # binary16 and bfloat16; one operand or both, the other one K-contiguous or not
    for f in by_words:
        assert _longest_run_of_loads(forms[f]) >= 16, f

"""gemm_stage_kernel on rows that need no straightening holds nothing of what straightened rows need (what runs once costs by its
length): its instructions are those that it had before there was such a form.  Seen in the code built."""
from code_util import kernels

# both operands K-contiguous, only A, only B, neither; with the other form's condition in it the first and third had 9 .. 18 more
MOST = {("64", "64"): (1934, 1945, 1944, 1789), ("64", "128"): (2647, 2630, 2634, 2495), ("128", "64"): (2736, 2724, 2720, 2582),
        ("128", "128"): (4018, 4027, 4028, 3891)}


def test_plain_rows_carry_nothing_of_straightened_ones():
    forms = kernels("gemm_stage_kernel")
    plain = {f: code for f, code in forms.items() if not f[-1]}
    assert len(plain) == 2 * 4 * 4 and len(forms) - len(plain) == 2 * 4 * 3
    for f, code in plain.items():
        assert len(code) <= MOST[f[1:3]][2 * (not f[6]) + (not f[7])], (f, len(code))

"""The selection prices the kernel that the launch will run: 16-bit products whose best tile runs the stage kernel on operands that
the caches hold.  It priced that kernel above the other one of the same tile there, and took another tile or more slices."""
import pytest

import paper_2003_06324_amd as g

R, C = g.ROW_MAJOR, g.COL_MAJOR


@pytest.mark.parametrize("M,N,K,align,la,lb,pick", [
    (2320, 878, 626, 4, C, R, "t128x128:s1"),    # 12.9 us with t64x64:s1, 11.3 with this
    (1176, 1676, 840, 8, C, R, "t128x128:s1"),   # 14.0 with t64x64:s1, 10.6
    (448, 832, 1856, 16, C, R, "t64x64:s1"),     # 11.3 in two slices, 8.5
    (1152, 256, 1728, 16, R, R, "t64x64:s1"),    # 10.7 in two slices, 8.4
])
def test_picks(M, N, K, align, la, lb, pick):
    assert g.query_config(2, M, N, K, align, la, lb) == pick

"""What a call pays for the selection where its shape is not among the kept picks: of the order of the query that finds it kept."""
import time

import paper_2003_06324_amd as g


def _microseconds(shapes):
    best = 1e9
    for _ in range(12):
        t = time.perf_counter()
        for M, N, K in shapes:
            g.query_config(2, M, N, K, 16, g.ROW_MAJOR, g.COL_MAJOR)
        best = min(best, time.perf_counter() - t)
    return best / len(shapes) * 1e6


def test_a_new_shape_costs_little():
    g.force_config(None)
    g.tune_clear()
    shapes = [(800 + 8 * i, 904 + 8 * (7 * i % 300), 1600 + 64 * (i % 37)) for i in range(500)]
    kept = _microseconds(shapes[:1] * len(shapes))
    new = _microseconds(shapes)
    # (0.2; 1.6 with every tile and slice count evaluated)
    assert new - kept < 0.6 * kept, (new, kept)

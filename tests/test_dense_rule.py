"""Which schedules the forward pools on the matrix cores (no GPU): the rule on
sizes and counts, at counts of real rigs on both sides of each of its lines.
"""

import pytest

from _sched import dense_forward


def _shape(B, H, W, D, X, C, N=6, Z=1):
    return dict(B=B, N=N, D=D, H=H, W=W, C=C, X=X, Y=X, Z=Z)


# (samples, rows, columns, bins, cells, channels), kept points, occupied cells, slots
@pytest.mark.parametrize("size,counts,dense", [
    ((1, 40, 100, 118, 128, 80), (1393768, 15656, 24297), True),
    ((4, 40, 110, 118, 256, 80), (6452079, 176206, 102354), True),
    ((1, 16, 44, 59, 128, 64), (130056, 9716, 2618), False),       # 10 points a segment
    # bins finer than the cells, segments that see most of a strip's pixels
    ((1, 40, 100, 472, 64, 80), (5543844, 3948, 15466), True),
    ((1, 16, 44, 472, 64, 80), (1024442, 3942, 3492), True),
    ((8, 4, 352, 472, 128, 80), (27921388, 125820, 132820), True),
    # and few of them
    ((4, 2, 100, 944, 128, 80), (3964188, 62872, 26873), False),
    ((4, 4, 100, 944, 64, 80), (7928376, 15799, 12145), False),
    ((4, 1, 100, 944, 64, 80), (1982094, 15799, 7355), False),
    ((1, 4, 100, 472, 64, 64), (991752, 3948, 3096), False),
    # low images, grids fine for their strips
    ((1, 4, 100, 236, 128, 80), (496348, 15694, 8032), False),
    ((4, 8, 44, 236, 128, 80), (1348230, 52513, 21311), False),
    ((1, 2, 352, 118, 64, 80), (437648, 3940, 4283), True),
])
@pytest.mark.parametrize("half", [False, True])
def test_rule_at_counts_of_real_rigs(size, counts, dense, half):
    assert dense_forward(_shape(*size), *counts, half=half) == dense


def test_rule_needs_strips_that_a_byte_numbers():
    counts = (400000, 5000, 5000)
    assert dense_forward(_shape(1, 16, 44, 118, 128, 36), *counts)       # 224 pixels
    assert not dense_forward(_shape(1, 16, 44, 118, 128, 32), *counts)   # 256


def test_rule_of_narrow_float16_rows():
    """Their walk costs more, so emptier tables pay."""
    counts = (124840, 989, 1031)
    assert dense_forward(_shape(1, 4, 100, 59, 32, 40), *counts, half=True)
    assert not dense_forward(_shape(1, 4, 100, 59, 32, 40), *counts)
    assert not dense_forward(_shape(1, 4, 100, 472, 64, 64), 991752, 3948, 3096, half=True)

"""The brick order of the FP64 global table, restated from its definition and checked on the CPU: 2 x 2 x 4 entries of
(hi, mid, lo) to a 128-byte brick, bricks counted row by row.  The closed forms the kernels index by must give every
entry a place of its own inside the allocation, and 32-bit byte offsets up to the largest table radius."""
import numpy as np
import pytest


def brick_count(H):
    return (H + 1) * (H + 3) * (2 * H + 1) // 24


def offset(hi, mid, lo):
    b_hi = 128 * brick_count(hi // 2) + 64 * (hi & 1)
    b_mid = 128 * ((mid // 2 + 1) ** 2 // 4) + 32 * (mid & 1)
    q = 4 * lo                                      # the kernels' lo is quantised: 4 lo
    return b_hi + b_mid + 2 * q + 96 * (q >> 4)


def test_counts_are_the_rows_before():
    total = 0
    for H in range(601):
        assert brick_count(H) == total
        row = 0
        for M in range(H + 1):
            assert (M + 1) ** 2 // 4 == row
            row += M // 2 + 1                       # lo <= 2 M + 1
        total += row


@pytest.mark.parametrize("R", [47, 48, 60, 61, 121])
def test_every_entry_has_its_own_place(R):
    hi, mid, lo = (a.ravel() for a in np.meshgrid(*[np.arange(R + 1)] * 3, indexing="ij"))
    k = (lo <= mid) & (mid <= hi)
    o = offset(hi[k], mid[k], lo[k])
    assert len(np.unique(o)) == k.sum() and (o % 8 == 0).all()
    assert o.min() == 0 and o.max() + 8 <= 8 * 16 * brick_count(R // 2 + 1)
    # a brick holds 2 x 2 x 4 neighbours
    b = o // 128
    same = np.lexsort((lo[k], mid[k], hi[k], b))
    first = np.searchsorted(b[same], b[same])
    for v, w in ((hi[k], 2), (mid[k], 2), (lo[k], 4)):
        assert (v[same] // w == (v[same] // w)[first]).all()


def test_offsets_fit_32_bits_at_the_largest_radius():
    assert offset(1200, 1200, 1200) < 2 ** 32

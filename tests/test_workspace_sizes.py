"""Workspace of prefill shapes where a plan with more key splits is estimated no
faster than one with fewer, by a block shape of half the rows (host side only)."""
import pytest

from paper_2608_19920_amd import h2o as H

MIB = 1 << 20


@pytest.mark.parametrize("shape,most", [
    # B, Hq, Hkv, T, M, d: unsplit 25 and 46 MiB (column partials, statistics, scores);
    # the O partials of two splits alone would be 128 and 145
    ((3, 28, 4, 1563, 3856, 128), 30 * MIB),
    ((5, 16, 8, 1856, 7416, 128), 50 * MIB),
], ids=str)
def test_equal_plans_take_the_smaller_workspace(shape, most):
    assert 0 < H.h2o_workspace_bytes(*shape, 1) <= most

"""The single-precision cell sort on both sides of the rule (slots squared over
cells) from which the scatter orders each block's particles in LDS, against a
stable sort on the CPU."""
import math

import pytest

from test_gpu_sort_ordered import G, test_sort_in_single_precision as sorts  # noqa: F401

pytestmark = pytest.mark.gpu

EDGE = math.isqrt(2 ** 26 * 96 * 57 - 1) + 1  # the fewest slots of the ordered form on that test's grid


@pytest.mark.parametrize("order", ["random", "near"])
@pytest.mark.parametrize("n", [EDGE - 1, EDGE, 1024 * (EDGE // 1024 + 1)])
def test_sorts_around_the_rule(G, n, order):
    sorts(G, n, order)

"""The automatic chunk size of the searches (no GPU): grids where the measured
best differs between the two kernels or where one size is clearly slower."""

import pytest

from paper_2103_10453_amd import instances as gen
from paper_2103_10453_amd import plse as P


def _choice(n, ratio, kernel, variant=0):
    h = P.plse_create(gen.random_greedy(n, ratio, 7))
    try:
        P.plse_set_param(h, "plits_kernel", kernel)
        P.plse_set_param(h, "variant", variant)
        return P.plse_get_param(h, "plits_kernel"), P.plse_get_param(h, "slots_per_lane")
    finally:
        P.plse_destroy(h)


# us of 600 to 2500 iterations, 4096 (or 256) side by side, with the size named
# and with the other candidate
@pytest.mark.parametrize("n,ratio,size", [
    (10, 0.4, 2),   # 3256, 4: 3434, 8: 5323
    (16, 0.7, 2),
    (20, 0.6, 4),   # 4231, 2: 4612
    (24, 0.4, 4),   # 5194, 8: 7633
    (24, 0.7, 4),   # 4592, 2: 4874
    (40, 0.7, 4),   # 7793, 8: 11698
    (40, 0.8, 4),   # 6057, 2: 6404
    (32, 0.3, 8),   # 11109, 4: 12820
    (50, 0.5, 8),
    (80, 0.8, 4),   # 33782, 8: 41837
    (90, 0.8, 4),   # 59205, 8: 68845
])
def test_lds_resident_kernel(n, ratio, size):
    assert _choice(n, ratio, 2) == (2, size)


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("n,ratio,size", [
    (10, 0.4, 2),
    (16, 0.3, 4),
    (50, 0.5, 8),
    (70, 0.7, 8),
    (70, 0.8, 4),
    (28, 0.7, 4),   # 3996, 2: 4157
    (40, 0.7, 4),   # 4743, 8: 5173
    (80, 0.8, 4),   # depth 60: 1486, 8: 1618
    (90, 0.8, 4),   # depth 60: 1590, 8: 1762
])
def test_global_table_kernel(n, ratio, size, variant):
    assert _choice(n, ratio, 1, variant) == (1, size)

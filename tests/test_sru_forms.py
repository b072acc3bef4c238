"""Which XCDs the workgroups of a one-kernel SRU layer go to, asked of the library's rule compiled for the host."""
import pytest

from test_launch_grids import _compiled

RULE = """
#include "sru_forms.h"
#include <stdio.h>
int main()
{
    int B, L, n_in, n_h, layers, first_two, later_two;
    while (scanf("%d %d %d %d %d %d %d", &B, &L, &n_in, &n_h, &layers, &first_two, &later_two) == 7)
        printf("%d\\n", moe::sru_deals_channels(B, L, n_in, n_h, layers, first_two, later_two));
}
"""


@pytest.fixture(scope="module")
def deals(tmp_path_factory):
    ask = _compiled(tmp_path_factory, "sru_forms", RULE)
    return lambda *shape, two=(0, 0): bool(ask([list(shape) + list(two)])[0][0])


@pytest.mark.parametrize("shape", [
    (14, 18, 768, 512, 4), (9, 23, 768, 256, 10), (10, 58, 768, 256, 9),         # weights of a predictor past an XCD's L2, few rows
    (30, 41, 768, 1024, 4), (5, 1, 768, 1024, 4), (2, 23, 256, 1024, 4),
    (9, 16, 960, 512, 1), (3, 19, 1024, 768, 2), (7, 8, 512, 384, 4), (9, 11, 640, 768, 1),   # most of an L2, next to no rows
    (49, 66, 256, 1024, 3), (15, 182, 1536, 768, 1), (38, 255, 768, 1024, 3),    # weights of a layer past it: fetched again for every sequence
])
def test_few_rows_under_many_weights_are_dealt_by_channel(deals, shape):
    assert deals(*shape)
    assert not deals(8 * shape[0], *shape[1:])                                   # multiples of 8: whole sequences, as ever
    assert not deals(*shape, two=(1, 1))                                         # no layer in one kernel


@pytest.mark.parametrize("shape", [
    (12, 512, 256, 256, 4), (5, 777, 768, 256, 2), (6, 600, 256, 256, 4), (12, 260, 256, 256, 9), (10, 225, 256, 256, 2),   # rows outweigh them
    (1, 1, 768, 1024, 4), (2, 7, 768, 512, 4), (1, 300, 768, 256, 10),           # an XCD has a part of a sequence, whose weights fit
    (17, 40, 64, 128, 4), (5, 8, 512, 384, 4),                                   # all weights fit
    (7, 95, 128, 256, 10), (47, 31, 128, 512, 3),                                # nearly, and rows that count
])
def test_others_keep_their_sequences_together(deals, shape):
    assert not deals(*shape)

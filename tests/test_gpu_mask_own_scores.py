"""Prefill masks of k/bk up to 128 whose nodes hand on their own scores alone (first or last block as representative, and the centre with 64
channels and one scored row a block), up to the full table of 128 nodes, whose upper half holds those scores; and the centre beside them."""
import pytest

from tests.test_gpu_carried_scores_wide import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rep_pos", [0, 1, 2])
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("kb,bk,d,bq,hq,batch", [(128, 1, 64, 32, 1, 8), (64, 1, 64, 32, 3, 4), (128, 8, 128, 32, 1, 4), (125, 2, 128, 64, 1, 8),
                                                 (128, 1, 64, 32, 3, 180), (64, 1, 64, 16, 4, 120), (128, 2, 128, 32, 4, 110), (127, 4, 128, 32, 4, 100),
                                                 (128, 1, 128, 64, 3, 260), (33, 1, 64, 32, 4, 110)])
def test_indices(kb, bk, d, bq, hq, batch, page, rep_pos):
    check(kb, bk, d, hq, batch, 100, bq, page, rep_pos, 6)

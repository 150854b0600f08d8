"""Prefill attention with query tiles of every number of rows around 8, 16 and 32, from which more of the tile is loaded.

Every number is the block's own rows and the rows of a sequence's last block; local memory holds NaN patterns before each launch."""
import pytest

from paper_2406_09827_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bq", [1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 40, 48, 49, 64])
def test_rows_of_a_tile(bq, d, page):
    for q_len, k in ((bq + 1, 32), (2 * bq + bq // 2 + 1, 160)):   # (one key tile, and five; the last block has few rows)
        w = synth.Workload("rows", 2, 4, 2, d, q_len, 900, k, bq, 2, "bf16", rho=0.9, page_size=page, integer=True, seed=340 + bq)
        U.run_case(w)

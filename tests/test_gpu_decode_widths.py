"""Decode on either side of the line between sixteen and four waves per (sequence, head): 256 and 264 problems, block lists
from less than a stage of one wave to several stages of every wave, at every block width and head dim."""
import pytest
import torch

import paper_2406_09827_amd as hipattn
from paper_2406_09827_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [32, 33])
@pytest.mark.parametrize("bk,d,k,T,page", [
    (1, 128, 3, 90, 0),        # three keys: most waves have no stage
    (2, 64, 130, 1500, 16),    # 65 blocks: one block in the last stage
    (1, 64, 513, 1700, 0),     # k/bk = 513 (beyond the sixteen-wave mask kernel)
    (4, 128, 2048, 4000, 64),  # k/bk = 512
    (8, 64, 1024, 2600, 0),    # blocks walked in pieces
    (2, 128, 512, 2100, 64),
    (4, 64, 260, 900, 0),
    (2, 128, 128, 1300, 16),   # k/bk = 64: the largest of the smallest list
])
def test_few_and_more_problems(batch, bk, d, k, T, page):
    for integer in (True, False):
        w = synth.Workload("decode_widths", batch, 8, 2, d, 1, T, k, 1, bk, "bf16", rho=0.9, ragged=(1, T), page_size=page,
                           integer=integer, seed=811 + bk)
        units = [(b, h, 0) for b in (0, 1, 7, 18, batch - 1) for h in (0, 3, 7)]
        U.run_case(w, 0, units=units, n_sink=k % 5, n_window=T % 7)


@pytest.mark.parametrize("bk,d,k", [
    # the last block list that four waves take alone and the first of sixteen: mask estimation (2 k/bk branches against one
    # stage each of four waves), then attention (k/bk blocks, or pieces of four rows, against one stage each)
    (2, 128, 32), (2, 128, 34), (2, 128, 64), (2, 128, 66),
    (1, 64, 64), (1, 64, 65), (1, 64, 128), (1, 64, 129),
    (4, 128, 32), (4, 128, 36), (4, 128, 64), (4, 128, 68), (8, 128, 64), (8, 128, 72), (8, 64, 128), (8, 64, 136),
    # stages of four and of eight rows
    (2, 128, 256), (2, 128, 258), (2, 128, 514),
])
@pytest.mark.parametrize("page", [0, 16])
def test_short_block_lists(bk, d, k, page):
    for n_sink, n_window, b_sk in ((0, 0, 1), (1, 2, 1), (5, 30, 2 if bk > 1 else 1)):
        T = 6 * k + 41
        w = synth.Workload("decode_short", 9, 8, 2, d, 1, T, k, 1, bk, "bf16", rho=0.9, ragged=(k, T), page_size=page, integer=True, seed=821 + bk)
        U.run_case(w, 0, n_sink=n_sink, n_window=n_window, b_sk=b_sk)


@pytest.mark.parametrize("bk,d,k", [(1, 64, 20), (2, 128, 256), (4, 64, 900), (8, 128, 4096), (2, 64, 1200)])
def test_slices_beyond_32_bit_offsets(bk, d, k):
    # rows 512 KB apart: a slice of over 2 GB, on the sixteen-wave (12 problems) and the four-wave kernels.  Same indices as from
    # the packed keys.
    T, pitch, hq = max(4100, 4 * k // 3), 1 << 18, 4
    w = synth.Workload("wide_slice", 1, hq, 1, d, 1, T, k, 1, bk, "bf16", rho=0.9, integer=True, seed=831)
    K = synth.make_inputs(w, device="cuda", threads=4)["K"]
    far = torch.empty(T * pitch, dtype=torch.bfloat16, device="cuda").as_strided((1, 1, T, d), (T * pitch, T * pitch, pitch, 1))
    far.copy_(K)
    for batch in (3, 66):
        Q = torch.randn(batch, hq, 1, d, device="cuda", generator=torch.Generator(device="cuda").manual_seed(batch)).bfloat16()
        lens = torch.tensor([T - 7 * (i % 5) for i in range(batch)], dtype=torch.int32, device="cuda")
        for rep_pos in (0, 1):
            a, b = (hipattn.hip_mask_estimate(Q, x.expand(batch, 1, T, d), k, 1, bk, kv_lens=lens, rep_pos=rep_pos) for x in (K, far))
            assert torch.equal(a, b)

"""Prefill mask estimation on either side of the lines between its kernels: table sizes (k/bk of 128, 256, 512), query tiles,
head dims, a workgroup or a wave per work item, paged and contiguous keys, and the launch shapes for long contexts."""
import pytest
import torch

import paper_2406_09827_amd as hipattn
from paper_2406_09827_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("heads", [(4, 1), (6, 2)], ids=["g4", "g3"])
@pytest.mark.parametrize("k,bk,d,bq,rep_pos", [
    (128, 1, 128, 32, 0), (258, 2, 128, 64, 1), (256, 1, 64, 64, 2), (1028, 4, 64, 32, 0), (1024, 2, 128, 32, 2),
    (514, 1, 128, 64, 0), (64, 2, 64, 16, 0), (1032, 8, 128, 48, 1), (2048, 2, 128, 32, 0), (1030, 2, 64, 32, 1),
])
def test_table_sizes(k, bk, d, bq, rep_pos, heads, page):
    hq, hkv = heads
    for q_len in (3 * bq + 5, bq * -(-1540 // hq)):   # below and above the line between a workgroup and a wave per work item
        T = max(q_len, 7 * k + 3)
        w = synth.Workload("widths", 1, hq, hkv, d, q_len, T, k, bq, bk, "bf16", rho=0.9, page_size=page, integer=True, seed=300 + k)
        nqb = w.n_query_blocks
        assert hq * nqb <= 512 or hq * nqb > 1536
        units = [(0, h, qb) for h in (0, hq - 1) for qb in sorted({0, 1, nqb // 2, nqb - 1})]
        U.run_case(w, 0, units=units, rep_pos=rep_pos, b_sk=2 if bk == 8 else 1)
        U.run_case(synth.scaled(w, integer=False), 0, units=units[:3], rep_pos=rep_pos)


@pytest.mark.parametrize("T,d,hq,bq,bk", [
    (100_000, 128, 4, 32, 2), (100_000, 128, 3, 32, 2), (100_000, 128, 4, 64, 4),   # over 24 MB of keys: two workgroups to a compute unit
    (530_000, 128, 4, 32, 2), (530_000, 128, 3, 64, 4), (1_050_000, 64, 4, 32, 2),  # over 128 MB: one, with 64 channels two
])
def test_launch_shapes_of_long_contexts(T, d, hq, bq, bk):
    # How many workgroups share a compute unit follows the bytes of a kv head's keys, not how far apart they are stored, where the
    # host knows the lengths.  Same indices as with the lengths on the device, and as from keys stored among another head's.
    nqb = -(-1540 // hq)
    assert hq * nqb > 1536   # a wave per work item
    gen = torch.Generator(device="cuda").manual_seed(bk + d)
    K = torch.randn(1, 1, T, d, device="cuda", generator=gen).bfloat16()
    Q = torch.randn(1, hq, nqb * bq - 3, d, device="cuda", generator=gen).bfloat16()
    lens = torch.tensor([T], dtype=torch.int32, device="cuda")
    apart = torch.empty(1, T, 2, d, dtype=torch.bfloat16, device="cuda").permute(0, 2, 1, 3)[:, 1:]
    apart.copy_(K)
    for rep_pos in (0, 2):
        a = hipattn.hip_mask_estimate(Q, K, 256 * bk, bq, bk, rep_pos=rep_pos)
        b = hipattn.hip_mask_estimate(Q, K, 256 * bk, bq, bk, rep_pos=rep_pos, kv_lens=lens)
        c = hipattn.hip_mask_estimate(Q, apart, 256 * bk, bq, bk, rep_pos=rep_pos)
        assert torch.equal(a, b) and torch.equal(a, c)


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("d,bq,bk,k,n_sink,n_window", [
    (128, 32, 2, 512, 0, 0),      # the list of keys is full and never refilled
    (64, 32, 1, 545, 3, 0),       # one key in the eighteenth tile, then a sink tile
    (128, 16, 4, 1024, 40, 300),  # refills among selected, sink and window tiles
    (64, 64, 8, 2048, 0, 70),
    (128, 48, 16, 768, 16, 1),
])
def test_key_lists_and_waves_per_item(d, bq, bk, k, n_sink, n_window, page):
    # four, two and one wave per (head, query tile): up to 512 of them, up to 1024, more
    tiles = (bq + 31) // 32
    for items in (60, 513, 1032):
        hq = 8
        q_len = -(-items // (hq * tiles)) * bq - 3
        T = max(q_len, 3 * k) + 17
        w = synth.Workload("lists", 1, hq, 2, d, q_len, T, k, bq, bk, "bf16", rho=0.9, page_size=page, integer=False, seed=320 + bk)
        nqb = w.n_query_blocks
        units = [(0, h, qb) for h in (0, 5) for qb in sorted({0, nqb // 2, nqb - 1})]
        U.run_case(w, 0, units=units, n_sink=n_sink, n_window=n_window)
    # a prefix shorter than k: the list ends early
    w = synth.Workload("short", 1, 8, 2, d, k, k, k, bq, bk, "bf16", rho=0.9, page_size=page, integer=True, seed=330)
    U.run_case(w, 0, units=[(0, 0, 0), (0, 7, 1), (0, 3, w.n_query_blocks - 1)], n_sink=n_sink, n_window=n_window)


@pytest.mark.parametrize("T", [4194301, 4194303])
def test_last_keys_of_a_slice_of_four_gigabytes(T):
    # rows 1024 bytes apart: the longest slice whose rows 32-bit lane offsets reach, and one that takes 64-bit addresses.  Rows
    # that attend to the last keys, from blocks at the front and the back of the context, against plain attention.
    d, bq, bk, kb, pitch = 128, 32, 2, 24, 512
    gen = torch.Generator(device="cuda").manual_seed(5)
    blocks = torch.cat([torch.arange(4), torch.tensor([1000, 2 ** 20]), torch.arange(kb - 6) + (T - 1) // bk - (kb - 7)]) * bk
    rows = (blocks[:, None] + torch.arange(bk)).flatten()
    rows = rows[rows < T].cuda()
    K, V = (torch.empty(T * pitch, dtype=torch.bfloat16, device="cuda").as_strided((1, 1, T, d), (T * pitch, T * pitch, pitch, 1)) for _ in range(2))
    for x in (K, V):
        x[0, 0, 0] = 0
        x[0, 0, rows] = torch.randn(len(rows), d, device="cuda", generator=gen).bfloat16()
    Q = torch.randn(1, 4, bq, d, device="cuda", generator=gen).bfloat16()
    idx = blocks.int().cuda().expand(1, 4, 1, kb).contiguous()
    out = hipattn.hip_sparse_attn(Q, K, V, idx, kb * bk, bq, bk)[0].double()
    x = Q[0].double() @ K[0, 0, rows].double().T * d ** -0.5
    x = x.masked_fill(rows[None, :] > torch.arange(T - bq, T, device="cuda")[:, None], float("-inf"))
    ref = torch.softmax(x, -1) @ V[0, 0, rows].double()
    assert float((out - ref).abs().max()) <= 2e-2   # (outputs below 4: see gpu_util)

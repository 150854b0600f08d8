"""Rounds in which branches keep scores of earlier rounds: nodes of one to four blocks, in every order in which lengths can halve.

Contexts from a few blocks above k/bk up to twenty times as long, so that the initial nodes take every length from 1 to 20 with
every kind of remainder; scores that drive the search to the left only (a node's first block was then never scored), to the
right only (it always was), and integers with many ties.  Indices equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2406_09827_amd as hipattn
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def keys(kind, rng, T, d):
    K = torch.zeros(T, d)
    if kind == "integers":
        return torch.from_numpy(rng.integers(-4, 5, (T, d)).astype(np.float32)) / 8
    K[:, 0] = torch.from_numpy({"left": -np.arange(T), "right": np.arange(T), "noise": rng.standard_normal(T)}[kind].astype(np.float32))
    return K


def queries(kind, rng, shape):
    Q = torch.zeros(shape)
    Q[..., 0] = 1.0
    return torch.from_numpy(rng.integers(-4, 5, shape).astype(np.float32)) / 8 if kind == "integers" else Q


def paged(K, page, rng):
    # keys [T, d] as a pool of pages in random order, and the page table of one sequence
    T, d = K.shape
    n = -(-T // page)
    order = torch.from_numpy(rng.permutation(n))
    pool = torch.zeros(n, 1, page, d, dtype=K.dtype)
    pool[order] = torch.nn.functional.pad(K, (0, 0, 0, n * page - T)).view(n, 1, page, d)
    return pool.cuda(), order.int().cuda()


@pytest.mark.parametrize("rep_pos", [0, 1, 2])
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("kb,bk,d,bq,hq,few", [(16, 2, 128, 16, 4, False), (16, 1, 64, 33, 3, False), (24, 4, 64, 16, 1, True), (17, 2, 128, 64, 1, True)],
                         ids=["wave_shared", "wave_two_tiles", "workgroup", "workgroup_two_tiles"])
def test_prefill(kb, bk, d, bq, hq, few, page, rep_pos):
    T = 20 * kb * bk
    nqb = T // bq + 1
    batch = 1 if few else -(-1540 // (hq * nqb))   # a workgroup or a wave per work item
    T = nqb * bq - 3
    rng = np.random.default_rng(kb + bk)
    for kind in ("integers", "left", "right", "noise"):
        K = keys(kind, rng, T, d).bfloat16()
        Q = queries(kind, rng, (hq, T, d)).bfloat16()
        kw, Kg = {}, K[None, None].cuda().expand(batch, 1, T, d).contiguous()
        if page:
            Kg, table = paged(K, page, rng)
            kw = dict(page_table=table.expand(batch, len(table)).contiguous(), max_kv_len=T)
        idx = torch.full((batch, hq, nqb, kb), U.UNWRITTEN, dtype=torch.int32, device="cuda")
        hipattn.hip_mask_estimate(Q[None].cuda().expand(batch, hq, T, d).contiguous(), Kg, kb * bk, bq, bk, rep_pos=rep_pos, indices=idx, **kw)
        p = oracle.Problem(1, hq, 1, d, T, T, kb * bk, bq, bk, n_threads=8, rep_pos=rep_pos)
        ref = oracle.mask_estimate(p, Q[None].float().numpy(), K[None, None].float().numpy())
        got = idx.cpu().numpy()
        assert (got == ref).all(), (kind, np.argwhere(got != ref)[:3])


@pytest.mark.parametrize("rep_pos", [0, 1, 2])
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("kb,bk,d,hq,batch", [(24, 2, 128, 2, 124), (72, 1, 64, 1, 250), (16, 4, 64, 2, 160), (24, 8, 128, 3, 90), (16, 2, 64, 8, 1030), (20, 1, 128, 8, 2050)],
                         ids=["sixteen_waves", "sixteen_waves_narrow", "four_waves", "four_waves_wide", "one_wave", "one_wave_128"])
def test_decode(kb, bk, d, hq, batch, page, rep_pos):
    # every sequence has a length of its own, of the same keys
    T = 20 * kb * bk
    rng = np.random.default_rng(kb + 7 * bk)
    lens = np.sort(rng.integers(kb * bk + 1, T + 1, batch)).astype(np.int32)
    lens[-1] = T
    for kind in ("integers", "left", "right", "noise"):
        K = keys(kind, rng, T, d).bfloat16()
        Q = queries(kind, rng, (batch, hq, 1, d)).bfloat16()
        kw, Kg = dict(kv_lens=torch.from_numpy(lens).cuda(), max_kv_len=T), K[None, None].cuda().expand(batch, 1, T, d)
        if page:
            Kg, table = paged(K, page, rng)
            kw["page_table"] = table.expand(batch, len(table)).contiguous()
        idx = torch.full((batch, hq, 1, kb), U.UNWRITTEN, dtype=torch.int32, device="cuda")
        hipattn.hip_mask_estimate(Q.cuda(), Kg, kb * bk, 1, bk, rep_pos=rep_pos, indices=idx, **kw)
        some = np.unique(rng.integers(0, batch, 60))
        p = oracle.Problem(len(some), hq, 1, d, 1, T, kb * bk, 1, bk, n_threads=8, rep_pos=rep_pos, kv_lens=lens[some].copy())
        ref = oracle.mask_estimate(p, Q[some].float().numpy(), np.broadcast_to(K.float().numpy(), (len(some), 1, T, d)).copy())
        got = idx.cpu().numpy()[some]
        assert (got == ref).all(), (kind, np.argwhere(got != ref)[:3])


@pytest.mark.parametrize("rep_pos", [0, 1, 2])
@pytest.mark.parametrize("dtype,kb,bk,d,bq", [("fp32", 16, 2, 64, 16), ("fp32", 70, 1, 128, 48), ("fp32", 17, 5, 64, 32), ("bf16", 16, 3, 128, 16)])
def test_any_shape(dtype, kb, bk, d, bq, rep_pos):
    T = 20 * kb * bk - 3
    rng = np.random.default_rng(kb + 5 * bk)
    for kind in ("integers", "left", "right", "noise"):
        dt = torch.float32 if dtype == "fp32" else torch.bfloat16
        K, Q = keys(kind, rng, T, d).to(dt)[None, None], queries(kind, rng, (1, 2, T, d)).to(dt)
        idx = torch.full((1, 2, -(-T // bq), kb), U.UNWRITTEN, dtype=torch.int32, device="cuda")
        hipattn.hip_mask_estimate(Q.cuda(), K.cuda(), kb * bk, bq, bk, rep_pos=rep_pos, indices=idx)
        ref = oracle.mask_estimate(oracle.Problem(1, 2, 1, d, T, T, kb * bk, bq, bk, n_threads=8, rep_pos=rep_pos), Q.float().numpy(), K.float().numpy())
        got = idx.cpu().numpy()
        assert (got == ref).all(), (kind, np.argwhere(got != ref)[:3])

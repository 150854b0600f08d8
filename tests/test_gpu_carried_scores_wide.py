"""Scores of earlier rounds in the kernels of more than 64 nodes: every number of keys a lane, of one, four and sixteen waves a problem
or work item, contiguous and over pages, with all three representatives.

Sequences of their own lengths over the same keys, from a few blocks above k/bk up to twenty times as many, and searches driven left,
right, at random and through ties.  Indices equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2406_09827_amd as hipattn
from tests import gpu_util as U
from tests.test_gpu_carried_scores import keys, paged, queries

pytestmark = pytest.mark.gpu


def check(kb, bk, d, hq, batch, q_len, bq, page, rep_pos, n_sampled):
    T = 20 * kb * bk
    rng = np.random.default_rng(kb + 7 * bk)
    lens = np.sort(rng.integers(kb * bk + q_len, T + 1, batch)).astype(np.int32)
    lens[-1] = T
    nqb = -(-q_len // bq)
    for kind in ("integers", "left", "right", "noise"):
        K = keys(kind, rng, T, d).bfloat16()
        Q = queries(kind, rng, (batch, hq, q_len, d)).bfloat16()
        kw, Kg = dict(kv_lens=torch.from_numpy(lens).cuda(), max_kv_len=T), K[None, None].cuda().expand(batch, 1, T, d)
        if page:
            Kg, table = paged(K, page, rng)
            kw["page_table"] = table.expand(batch, len(table)).contiguous()
        idx = torch.full((batch, hq, nqb, kb), U.UNWRITTEN, dtype=torch.int32, device="cuda")
        hipattn.hip_mask_estimate(Q.cuda(), Kg, kb * bk, bq, bk, rep_pos=rep_pos, indices=idx, **kw)
        some = np.unique(np.append(rng.integers(0, batch, n_sampled), batch - 1))
        p = oracle.Problem(len(some), hq, 1, d, q_len, T, kb * bk, bq, bk, n_threads=8, rep_pos=rep_pos, kv_lens=lens[some].copy())
        ref = oracle.mask_estimate(p, Q[some].float().numpy(), np.broadcast_to(K.float().numpy(), (len(some), 1, T, d)).copy())
        got = idx.cpu().numpy()
        assert (got != U.UNWRITTEN).all(), kind
        assert (got[some] == ref).all(), (kind, np.argwhere(got[some] != ref)[:3])


@pytest.mark.parametrize("rep_pos", [0, 1, 2])
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("kb,bk,d,hq,batch", [(130, 1, 128, 2, 100), (300, 1, 64, 1, 250), (300, 8, 128, 1, 40),
                                              (72, 2, 128, 3, 90), (130, 4, 64, 2, 140), (300, 1, 128, 2, 130), (1024, 1, 64, 1, 260),
                                              (72, 2, 64, 8, 1030), (130, 1, 64, 8, 1030), (300, 2, 64, 8, 1030)],
                         ids=["sixteen_130", "sixteen_300", "sixteen_300_wide", "four_72", "four_130", "four_300", "four_1024", "one_72", "one_130", "one_300"])
def test_decode(kb, bk, d, hq, batch, page, rep_pos):
    check(kb, bk, d, hq, batch, 1, 1, page, rep_pos, 30 if kb < 300 else 16 if kb < 1024 else 8)


@pytest.mark.parametrize("rep_pos", [0, 1, 2])
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("kb,bk,d,bq,hq,batch", [(130, 2, 128, 32, 1, 8), (300, 1, 64, 64, 2, 6), (300, 4, 128, 64, 1, 6), (1024, 1, 64, 32, 1, 3),
                                                 (130, 2, 128, 64, 4, 200), (300, 1, 64, 32, 3, 180), (300, 2, 128, 64, 4, 200), (1024, 1, 64, 16, 4, 80)],
                         ids=["workgroup_130", "workgroup_300", "workgroup_300_two_tiles", "workgroup_1024",
                              "wave_130_two_tiles", "wave_300", "wave_300_two_tiles", "wave_1024"])
def test_prefill(kb, bk, d, bq, hq, batch, page, rep_pos):
    check(kb, bk, d, hq, batch, 100, bq, page, rep_pos, 6 if kb < 300 else 3 if kb < 1024 else 1)

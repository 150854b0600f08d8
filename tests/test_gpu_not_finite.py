"""Mask estimation of inputs that are not finite: which blocks are kept is open, but every query block gets k/bk ascending blocks
of its own prefix.  (Block positions find their pages through the table: a position that is none would read past it.)"""
import pytest
import torch

import paper_2406_09827_amd as hipattn
from paper_2406_09827_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _bf16_bits(x, rows, bits):
    x.view(torch.int16)[rows] = bits


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("k,bk,d", [(120, 1, 64), (400, 2, 128), (1200, 4, 128), (600, 1, 64)])
@pytest.mark.parametrize("shape", ["prefill", "prefill_few", "decode", "decode_four_waves"])
def test_indices_stay_valid(shape, k, bk, d, page):
    batch, hq, hkv, q_len, bq = {"prefill": (1, 8, 2, 800, 2), "prefill_few": (2, 4, 2, 150, 64), "decode": (3, 8, 2, 1, 1),
                                 "decode_four_waves": (40, 8, 2, 1, 1)}[shape]
    T = 5 * k + 37
    w = synth.Workload("nan", batch, hq, hkv, d, min(q_len, T), T, k, bq, bk, "bf16", rho=0.9, page_size=page, ragged=(2 * k + 50, T) if batch > 1 else None,
                       seed=801)
    units = [(b, h, qb) for b in range(batch) for h in range(hq) for qb in range(w.n_query_blocks)]
    for what in ("queries", "most keys", "infinite keys"):
        x = synth.make_inputs(w, device="cuda", threads=4)
        if what == "queries":
            _bf16_bits(x["Q"], ..., -64)
        else:
            rows = torch.rand(x["K"].shape[:3], generator=torch.Generator().manual_seed(k)) < 0.9
            _bf16_bits(x["K"], rows.cuda(), -64 if what == "most keys" else -128)   # -NaN, -inf (times a query of either sign)
        for rep_pos, ens in ((0, 0), (2, 0), (0, 1)):
            U.probes.poison_lds(0x7FFF7FFF)
            idx = torch.full((batch, hq, w.n_query_blocks, w.kb), U.UNWRITTEN, dtype=torch.int32, device="cuda")
            hipattn.hip_mask_estimate(x["Q"], x["K"], w.k, bq, bk, kv_lens=x["kv_lens"], page_table=x["page_table"],
                                      max_kv_len=U._max_len(w, x), rep_pos=rep_pos, ens_sample=ens, ens_seed=3, ens_r=2.0, indices=idx)
            U.check_indices_valid(w, x, idx.cpu().numpy().reshape(-1, w.kb), units)

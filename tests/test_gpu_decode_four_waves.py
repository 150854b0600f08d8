"""The options of mask estimation on the decode kernels with four waves a (sequence, head), which serve 257 to 8192 problems:
sampling stride and representative (scores carried from round to round), ensemble samples (the perturbed round), top-r
channels, the token bank with its maps of pages read, and a captured graph, for every number of keys a lane holds."""
import pytest
import torch

import paper_2406_09827_amd as hipattn
from paper_2406_09827_amd import synth
from tests import gpu_util as U
from tests.test_gpu_ensemble import _samples_match

pytestmark = pytest.mark.gpu
UNITS = [(b, h, 0) for b in (0, 3, 17, 32) for h in (0, 3, 7)]


def _workload(kb, bk, integer=True, d=128, page=0, T=0):
    T = T or 7 * kb * bk + 53
    return synth.Workload("dec4", 33, 8, 2, d, 1, T, kb * bk, 1, bk, "bf16", rho=0.9, ragged=(T // 9, T), page_size=page, integer=integer, seed=841 + kb)


@pytest.mark.parametrize("kb", [64, 128, 256, 512])
@pytest.mark.parametrize("bk,b_sk,rep_pos,page", [(2, 2, 0, 0), (4, 2, 1, 16), (8, 2, 2, 0), (2, 1, 1, 0), (1, 1, 2, 16)])
def test_scoring_options(kb, bk, b_sk, rep_pos, page):
    for integer in (True, False):
        U.run_case(_workload(kb, bk, integer, 64 if bk == 4 else 128, page), 0, units=UNITS, b_sk=b_sk, rep_pos=rep_pos, n_sink=3, n_window=21)


@pytest.mark.parametrize("kb", [64, 128, 256, 512])
def test_ensemble_samples_and_top_r(kb):
    _samples_match(_workload(kb, 2), 3, 31, 5.0, units=UNITS)
    _samples_match(_workload(kb, 2, page=16), 2, 32, 5.0, units=UNITS, rep_pos=2)
    U.run_case(_workload(kb, 2), 0, units=UNITS, top_r=24)


@pytest.mark.parametrize("kb", [64, 128, 256, 512])
def test_token_bank(kb):
    U.run_bank_case(_workload(kb, 1, page=16, T=3 * kb + 200), 0.5, n_sink=3, n_window=20, rep_pos=kb // 64 % 3)
    U.run_bank_case(_workload(kb, 2, page=16, T=5 * kb + 200), 0.3, b_sk=2)


@pytest.mark.parametrize("kb", [64, 128, 256, 512])
def test_replayed_from_a_graph(kb):
    w = _workload(kb, 2, page=16)
    x = synth.make_inputs(w, device="cuda", threads=4)
    idx = torch.empty((w.batch, w.n_q_heads, 1, w.kb), dtype=torch.int32, device="cuda")
    out = torch.empty_like(x["Q"])

    def step():
        kw = dict(kv_lens=x["kv_lens"], page_table=x["page_table"])
        hipattn.hip_mask_estimate(x["Q"], x["K"], w.k, w.bq, w.bk, indices=idx, rep_pos=1, **kw)
        hipattn.hip_sparse_attn(x["Q"], x["K"], x["V"], idx, w.k, w.bq, w.bk, out=out, n_sink=4, n_window=16, **kw)

    step()
    torch.cuda.synchronize()
    idx_ref, out_ref = idx.clone(), out.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        step()
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.current_stream().wait_stream(side)
    for r in range(3):
        idx.fill_(U.UNWRITTEN)
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(idx, idx_ref) and torch.equal(out, out_ref), f"replay {r}"

"""The top-k selection of a round on score distributions that its search handles differently: far-out scores, equal scores,
nearly equal ones, two clusters, heavy tails; for every number of keys a lane can hold, in each family of mask kernels.

Every query row is the first unit vector, so that a key's score is its first channel, exactly: indices equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2406_09827_amd as hipattn
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

SCORES = {
    "normal": lambda r, n: r.standard_normal(n),
    "one_far_out": lambda r, n: np.where(np.arange(n) == n // 3, 1e4, r.standard_normal(n)),
    "some_far_out": lambda r, n: np.where(r.random(n) < 0.01, 40.0, 1.0) * r.standard_normal(n),
    "heavy_tails": lambda r, n: np.sinh(6.0 * r.standard_normal(n)),
    "two_values": lambda r, n: np.where(r.random(n) < 0.5, 1.5, 0.25),
    "integers": lambda r, n: r.integers(-8, 9, n).astype(float),
    "a_third_equal": lambda r, n: np.where(r.random(n) < 0.33, 0.0625, r.standard_normal(n)),
    "constant": lambda r, n: np.full(n, -1.75),
    "nearly_constant": lambda r, n: 1.0 + r.integers(0, 3, n) / 128.0,
    "two_clusters": lambda r, n: r.standard_normal(n) + np.where(r.random(n) < 0.5, 20.0, 0.0),
    "falling": lambda r, n: -np.arange(n, dtype=float),
}


@pytest.mark.parametrize("kb", [40, 64, 100, 128, 200, 256, 500, 900])
@pytest.mark.parametrize("kernel", ["decode", "decode_four_waves", "prefill", "prefill_few", "any_shape_fp32"])
def test_selection_on_score_distributions(kernel, kb):
    T = 5 * kb + 77
    dtype = torch.float32 if kernel == "any_shape_fp32" else torch.bfloat16
    q_len, bq, hq, batch, d = {"decode": (1, 1, 4, 1, 64), "decode_four_waves": (1, 1, 4, 66, 64), "prefill": (520, 1, 4, 1, 64),
                               "prefill_few": (70, 64, 1, 1, 128), "any_shape_fp32": (70, 32, 1, 1, 64)}[kernel]
    q_len = min(q_len, T)
    rng = np.random.default_rng(kb)
    for name, scores in SCORES.items():
        K = torch.zeros(batch, 1, T, d)
        for b in (0, batch - 1):
            K[b, 0, :, 0] = torch.from_numpy(scores(rng, T))
        K = K.to(dtype)
        Q = torch.zeros(batch, hq, q_len, d, dtype=dtype)
        Q[..., 0] = 1.0
        nqb = -(-q_len // bq)
        for rep_pos, b_sq in ((0, 1), (2, max(1, bq // 2))):  # (sampled rows: branches of -inf near the end)
            idx = torch.full((batch, hq, nqb, kb), U.UNWRITTEN, dtype=torch.int32, device="cuda")
            hipattn.hip_mask_estimate(Q.cuda(), K.cuda(), kb, bq, 1, rep_pos=rep_pos, b_sq=b_sq, indices=idx)
            p = oracle.Problem(batch, hq, 1, d, q_len, T, kb, bq, 1, n_threads=8, rep_pos=rep_pos, b_sq=b_sq)
            units = np.array([(b, h, qb) for b in (0, batch - 1) for h in (0, hq - 1) for qb in sorted({0, nqb // 2, nqb - 1})], dtype=np.int32)
            ref = oracle.mask_estimate_units(p, Q.float().numpy(), K.float().numpy(), units)
            got = idx.cpu().numpy()[units[:, 0], units[:, 1], units[:, 2]]
            assert np.array_equal(got, ref), (name, rep_pos, b_sq)

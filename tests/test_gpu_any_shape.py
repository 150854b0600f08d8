"""The any-shape kernels (fp32, and bf16 shapes outside the tuned kernels) where their tiles and lists have edges:
16-row query tiles, 8 KB key tiles with blocks that straddle them, list sizes around the instantiated ones, odd page sizes."""
import pytest
import torch
import oracle

from paper_2406_09827_amd import synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

CASES = [
    # T, k, bq, bk, d, page
    (200, 2, 16, 1, 64, 0),        # two nodes
    (700, 63, 17, 3, 128, 0),      # 3-row blocks (one per two tiles straddles), one query row in the second tile
    (900, 64 * 5, 15, 5, 64, 0),   # k/bk = 64: the largest of the smallest list
    (1000, 65 * 5, 33, 5, 128, 15),  # k/bk = 65, three query tiles, 15-token pages
    (2000, 256, 64, 1, 128, 0),    # k/bk = 256, four query tiles
    (2000, 257, 32, 1, 64, 24),    # k/bk = 257
    (2600, 1026, 48, 2, 128, 0),   # k/bk = 513
    (2500, 1024, 1, 1, 64, 0),     # k/bk = 1024, one query row per block
    (3000, 512, 16, 16, 128, 48),  # largest key block
]


@pytest.mark.parametrize("T,k,bq,bk,d,page", CASES)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("integer", [True, False], ids=["int", "normal"])
def test_tile_and_list_edges(T, k, bq, bk, d, page, dtype, integer):
    w = synth.Workload("any", 1, 2, 1, d, T, T, k, bq, bk, dtype, rho=0.9, integer=integer, page_size=page, seed=901)
    n = w.n_query_blocks
    units = [(0, h, qb) for h in range(2) for qb in sorted({0, n // 3, n // 2, n - 2, n - 1})]
    U.run_case(w, U.hipattn.FORCE_GENERIC, units=units, rep_pos=(T // 100) % 3, n_sink=T % 7, n_window=T % 40, min_agreement=0.99)


def _attention_by_rows(Q, K, V, idx, bq, bk, sm_scale, n_sink, n_window, finfo_max):
    """Plain attention in 64 bits over the keys that count for each row, one sequence; a logit that overflows the type is infinite."""
    hq, T, d = Q.shape
    g = hq // K.shape[0]
    out = torch.zeros(hq, T, d, dtype=torch.float64)
    for h in range(hq):
        for i in range(T):
            w0 = max(i + 1 - n_window, 0)
            keys = set(range(min(n_sink, w0))) | set(range(w0, i + 1))
            for first in idx[h, i // bq].tolist():
                keys |= {t for t in range(first, first + bk) if n_sink <= t < w0}
            keys = sorted(keys)
            if not keys:
                continue
            x = (K[h // g, keys] @ Q[h, i]) * sm_scale
            x[x > finfo_max] = float("inf")
            out[h, i] = torch.softmax(x, 0) @ V[h // g, keys]
    return out


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("bq,bk,d,n_sink,n_window", [(16, 2, 64, 0, 0), (32, 5, 128, 3, 0), (64, 4, 128, 5, 20), (15, 1, 64, 0, 9)])
@pytest.mark.parametrize("odd", ["value", "key", "logit"])
def test_infinities_and_nan_reach_the_rows_that_attend_to_them_only(dtype, bq, bk, d, n_sink, n_window, odd):
    # An infinite or NaN value, a NaN key and a logit that overflows: rows that attend to the key show it, as plain
    # attention does; the rows of the same block before the key, and rows that re-read it as padding, do not.
    T, kb, dev = 130, 6, "cuda"
    gen = torch.Generator().manual_seed(17 * bk + bq)
    dt = {"fp32": torch.float32, "bf16": torch.bfloat16}[dtype]
    Q, K, V = (torch.randn(1, n, T, d, generator=gen).to(dt) for n in (2, 1, 1))
    nqb = -(-T // bq)
    idx = torch.full((1, 2, nqb, kb), U.hipattn.SENTINEL, dtype=torch.int32)
    for h in range(2):
        for qb in range(nqb):
            own = (min((qb + 1) * bq, T) - 1) // bk  # the block of the last row, and earlier ones (never block 0)
            pick = torch.randperm(max(own - 1, 0), generator=gen)[:kb - 2] + 1
            blocks = sorted({own, 23 // bk if qb % 2 else own, *pick.tolist()})
            idx[0, h, qb, :len(blocks)] = torch.tensor(blocks, dtype=torch.int32) * bk
    bad = ([] if n_sink else [0]) + [23, 40, T - 2]  # (as a sink key 0 would count for every row)
    if odd == "value":
        for t, x in zip(bad[::-1], (float("inf"), float("nan"), float("-inf"), float("inf"))):
            V[0, 0, t, t % d] = x
    elif odd == "key":
        K[0, 0, bad] = float("nan")
    else:
        Q[0, :, 48:] = 1e25
        for i, t in enumerate(bad):  # (no two alike: which of two equal logits of 1e26 is larger is up to the rounding)
            K[0, 0, t] = 1e25 * (i + 1)
    out = U.hipattn.hip_sparse_attn(Q.to(dev), K.to(dev), V.to(dev), idx.to(dev), kb * bk, bq, bk, n_sink=n_sink, n_window=n_window,
                                    flags=U.hipattn.FORCE_GENERIC)[0].double().cpu()
    ref = _attention_by_rows(Q[0].double(), K[0].double(), V[0].double(), idx[0], bq, bk, d ** -0.5, n_sink, n_window, 3.4e38)
    fin = torch.isfinite(ref)
    assert bool((~fin).any()) and bool(fin.any())
    assert torch.equal(torch.isnan(out), torch.isnan(ref)) and torch.equal(out[~fin & ~torch.isnan(ref)], ref[~fin & ~torch.isnan(ref)])
    # fp32: logits of up to 6e25 (the overflow case) decide by their order alone; the others are below 10, see gpu_util
    assert float((out - ref)[fin].abs().max()) <= (1e-4 if dtype == "fp32" else 2e-2)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("bq,bk,d,page", [(16, 4, 64, 8), (32, 5, 128, 15), (33, 16, 64, 48)])
def test_blocks_across_pages(dtype, bq, bk, d, page):
    # entries that are no multiples of bk: a block may go on in the next logical page, which lies anywhere in the pool
    T, kb, dev = 200, 5, "cuda"
    gen = torch.Generator().manual_seed(31 * bk + d)
    dt = {"fp32": torch.float32, "bf16": torch.bfloat16}[dtype]
    Q, K, V = (torch.randn(1, n, T, d, generator=gen).to(dt) for n in (2, 1, 1))
    nqb, n_pages = -(-T // bq), -(-T // page)
    idx = torch.full((1, 2, nqb, kb), U.hipattn.SENTINEL, dtype=torch.int32)
    for h in range(2):
        for qb in range(nqb):
            seen = min((qb + 1) * bq, T)
            first = int(torch.randint(0, bk, (1,), generator=gen))
            starts = torch.arange(first, seen, bk)[torch.randperm(len(torch.arange(first, seen, bk)), generator=gen)[:kb]].sort().values
            idx[0, h, qb, :len(starts)] = starts.int()
    table = torch.randperm(n_pages, generator=gen).int()
    pools = []
    for X in (K, V):
        pool = torch.zeros(n_pages, 1, page, d, dtype=dt)
        for i in range(n_pages):
            n = min(page, T - i * page)
            pool[table[i], 0, :n] = X[0, 0, i * page:i * page + n]
        pools.append(pool.to(dev))
    out = U.hipattn.hip_sparse_attn(Q.to(dev), *pools, idx.to(dev), kb * bk, bq, bk, page_table=table[None].to(dev), max_kv_len=T,
                                    n_sink=2, n_window=3, flags=U.hipattn.FORCE_GENERIC)[0].double().cpu()
    ref = _attention_by_rows(Q[0].double(), K[0].double(), V[0].double(), idx[0], bq, bk, d ** -0.5, 2, 3, 3.4e38)
    assert float((out - ref).abs().max()) <= (1e-4 if dtype == "fp32" else 2e-2)


@pytest.mark.parametrize("T,k,bq,bk,d", [(1024, 128, 16, 2, 64), (2500, 512, 32, 2, 128), (900, 128, 64, 4, 128), (700, 60, 15, 3, 64)])
def test_fp32_attention_keeps_fp32_precision(T, k, bq, bk, d):
    # On the kernel's own indices, against 64 bits: products and sums of 32 bits differ by a few 2^-24 of logits below 10,
    # i.e. by less than 5e-6 in the norm; one of weights, probabilities or values in 16 bits would differ by 1e-3.
    w = synth.Workload("prec", 1, 2, 1, d, T, T, k, bq, bk, "fp32", rho=0.9, seed=931)
    x = synth.make_inputs(w, device="cuda", threads=4)
    idx = U.gpu_mask(w, x)
    out = U.gpu_attn(w, x, idx, n_sink=3, n_window=20).cpu().double()
    p = U.oracle_problem(w, x, n_sink=3, n_window=20)
    hx = U.host(x)
    units = oracle.all_units(p)
    ref = torch.from_numpy(oracle.sparse_attn_units(p, hx["Q"], hx["K"], hx["V"], units, idx.cpu().numpy().reshape(-1, w.kb), 0.0)).double()
    got = torch.zeros_like(ref)
    for u, (b, h, qb) in enumerate(units):
        n = min(bq, T - qb * bq)
        got[u, :n] = out[b, h, qb * bq:qb * bq + n]
        ref[u, n:] = 0
    assert float((got - ref).norm() / ref.norm()) <= 5e-6


@pytest.mark.parametrize("bq,d", [(16, 64), (16, 128), (32, 64), (32, 128), (64, 64), (64, 128)])
@pytest.mark.parametrize("scale,best", [(1.0, 1 + 2.0 ** -20), (2.0 ** -118, 1 + 2.0 ** -20), (1.0, float("inf"))], ids=["one", "smallest", "infinite"])
def test_fp32_scores_keep_fp32_range(bq, d, scale, best):
    # 100 keys, 64 kept in one round, so exactly the 64 largest scores: 63 of 4, one of `best`, 36 of 1 (before and behind it),
    # times a power of two: the scores are exact in fp32, and 1 + 2^-20 is above 1 at any scale.
    T, k, dev = 100, 64, "cuda"
    score = torch.ones(T)
    score[torch.arange(T) % 3 != 0] = 4.0  # 66 of them
    score[[1, 50, 97]] = 1.0
    score[33] = best
    K = torch.zeros(1, 1, T, d)
    K[0, 0, :, 5] = score * scale
    Q = torch.zeros(1, 1, bq, d)
    Q[..., 5] = 1.0
    idx = U.hipattn.hip_mask_estimate(Q.to(dev), K.to(dev), k, bq, 1).cpu().flatten()
    want = torch.nonzero(score > 1.0).flatten()
    assert len(want) == k and torch.equal(idx.sort().values.long(), want)


@pytest.mark.parametrize("bq,bk,d", [(16, 2, 64), (32, 4, 128)])
@pytest.mark.parametrize("scale", [2.0 ** -118, 2.0 ** 120])
def test_fp32_attention_keeps_fp32_range(bq, bk, d, scale):
    # the smallest and the largest values: the same bound as test_fp32_attention_keeps_fp32_precision
    T, kb, dev = 130, 6, "cuda"
    gen = torch.Generator().manual_seed(bq + d)
    Q, K, V = (torch.randn(1, n, T, d, generator=gen) for n in (2, 1, 1))
    V *= scale
    nqb = -(-T // bq)
    idx = torch.full((1, 2, nqb, kb), U.hipattn.SENTINEL, dtype=torch.int32)
    for qb in range(nqb):
        seen = -(-min((qb + 1) * bq, T) // bk)
        idx[0, :, qb, :min(kb, seen)] = torch.randperm(seen, generator=gen)[:kb].sort().values.int() * bk
    out = U.hipattn.hip_sparse_attn(Q.to(dev), K.to(dev), V.to(dev), idx.to(dev), kb * bk, bq, bk)[0].double().cpu()
    ref = _attention_by_rows(Q[0].double(), K[0].double(), V[0].double(), idx[0], bq, bk, d ** -0.5, 0, 0, 3.4e38)
    assert float((out - ref).norm() / ref.norm()) <= 5e-6


@pytest.mark.parametrize("bq,d", [(16, 64), (32, 128), (64, 128)])
@pytest.mark.parametrize("lost", ["all", "bits", "to zero"])
def test_fp32_scores_of_queries_at_the_end_of_the_range(bq, d, lost):
    # as above, with a score that only the low bits of a query of 2^-120 beside one of 1 set apart (keys of 2^120), with nothing but
    # such queries, and with subnormal queries, whose planes are 0
    T, k, dev, e = 100, 64, "cuda", -140 if lost == "to zero" else -120
    score = torch.ones(T)
    score[torch.arange(T) % 3 != 0] = 4.0  # 66 of them
    score[[1, 50, 97]] = 1.0
    K, Q = torch.zeros(1, 1, T, d), torch.zeros(1, 1, bq, d)
    K[0, 0, :, 6] = score * 2.0 ** 120
    Q[..., 5], Q[..., 6] = (1 + 2.0 ** -20 if lost != "to zero" else 2.0) * 2.0 ** e, 2.0 ** e
    K[0, 0, 33, 5:7] = torch.tensor([2.0 ** 120, 0.0])
    if lost == "bits":
        Q[..., 9] = 1.0
    idx = U.hipattn.hip_mask_estimate(Q.to(dev), K.to(dev), k, bq, 1).cpu().flatten()
    want = torch.nonzero((score > 1.0) | (torch.arange(T) == 33)).flatten()
    assert len(want) == k and torch.equal(idx.sort().values.long(), want)


@pytest.mark.parametrize("bq,bk,d", [(16, 2, 64), (32, 4, 128)])
@pytest.mark.parametrize("case", ["small channel", "smallest channel", "far behind", "large queries", "small queries"])
def test_fp32_attention_of_mixed_magnitudes(case, bq, bk, d):
    # All keys selected, every channel against 64 bits by itself.  The bound is that of test_fp32_attention_keeps_fp32_precision for
    # logits below 10; "far behind": a first key with values of 0 whose logit is ahead by 86, i.e. logits with errors of a few
    # 2^-24 * 86.
    T, dev = 130, "cuda"
    gen = torch.Generator().manual_seed(bq + d)
    Q, K, V = (torch.randn(1, n, T, d, generator=gen) for n in (2, 1, 1))
    V = V.abs() + 0.5
    bound = 5e-6
    if case in ("small channel", "smallest channel"):
        V[..., 5] *= 2.0 ** (-118 if case == "small channel" else -124)
    elif case == "far behind":
        K *= 0.1
        K[..., 7], K[0, 0, 0], V[0, 0, 0], Q[..., 7] = 0, 0, 0, d ** 0.5
        K[0, 0, 0, 7] = 86.0
        V *= 2.0 ** 30
        bound = 8 * 2.0 ** -24 * 86
    else:
        e = 120 if case == "large queries" else -120
        Q, K = Q * 2.0 ** e, K * 2.0 ** -e
    nqb, kb = -(-T // bq), -(-T // bk)
    idx = (torch.arange(kb, dtype=torch.int32) * bk).expand(1, 2, nqb, kb).contiguous()
    out = U.hipattn.hip_sparse_attn(Q.to(dev), K.to(dev), V.to(dev), idx.to(dev), kb * bk, bq, bk)[0].double().cpu()
    ref = _attention_by_rows(Q[0].double(), K[0].double(), V[0].double(), idx[0], bq, bk, d ** -0.5, 0, 0, 3.4e38)
    assert bool(((out - ref)[:, 1:].norm(dim=(0, 1)) <= bound * ref[:, 1:].norm(dim=(0, 1))).all())

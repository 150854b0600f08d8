"""Host-side check of the benchmark's branch count (no GPU): the branches of a search that no earlier round can have scored."""
import random

import pytest

import bench
from paper_2406_09827_amd import synth


def _branches_scored(rng, Tb, kb, rep_pos, direction):
    """One search over Tb blocks with survivors at random, or the leftmost / rightmost ones: the branches scored, where a block
    that any earlier round has scored keeps its score."""
    bounds = [(2 * j * Tb + kb) // (2 * kb) for j in range(kb + 1)]
    nodes, known, scored = list(zip(bounds, bounds[1:])), set(), 0
    while max(e - s for s, e in nodes) > 1:
        branches = [x for s, e in nodes for x in ((s, s + (e - s) // 2), (s + (e - s) // 2, e)) if x[1] > x[0]]
        blocks = {s + (e - s) // 2 if rep_pos == 0 else s if rep_pos == 1 else e - 1 for s, e in branches}
        scored += len(blocks - known)
        known |= blocks
        keep = sorted(rng.sample(range(len(branches)), kb)) if direction == 0 else range(kb) if direction < 0 else range(len(branches) - kb, len(branches))
        nodes = [branches[i] for i in keep]
    return scored


@pytest.mark.parametrize("rep_pos", [0, 1, 2])
def test_no_search_scores_fewer_branches_than_the_bench_counts(rep_pos):
    rng = random.Random(rep_pos)
    for kb in (1, 4, 7, 16):
        for Tb in range(kb, 70 * kb, 1 + kb // 3):
            least = bench.least_branches_scored(Tb, kb, rep_pos)
            got = [_branches_scored(rng, Tb, kb, rep_pos, direction) for direction in (0, 0, -1, 1)]
            assert least <= min(got), (Tb, kb, got)
            if Tb <= 2 * kb:
                assert least == min(got) == (Tb if Tb > kb else 0)   # one round: every block is a branch
    # 64 blocks a node: five full rounds, and with the centre representative nothing that the sixth would have to score
    assert bench.least_branches_scored(64 * 256, 256) == 2 * 256 * 5
    assert bench.least_branches_scored(64 * 256, 256, 2) == 256 * 2 + 256 * 5


def test_scored_bytes_are_fewer_than_the_rounds_name():
    for w in (synth.C2, synth.C3, synth.C4):
        least, named = bench.mask_scored_bytes(w, None), bench.mask_algorithmic_bytes(w, None)
        assert 0.6 * named < least < named


def test_counted_bytes_take_the_place_of_algorithmic_ones():
    c = {"hbm_algorithmic": {"frac": 0.92}, "hbm_counter": {"frac": 0.71}, "l2_fill_algorithmic": {"frac": 0.19}}
    assert bench.pick_roof(c) == "hbm_counter"
    assert bench.pick_roof({**c, "hbm_counter": None}) == "hbm_algorithmic"
    assert bench.pick_roof({**c, "l2_fill_algorithmic": {"frac": 0.8}}) == "l2_fill_algorithmic"

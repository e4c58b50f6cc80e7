"""The 64-bit filter's steps of 64 columns, scored two columns at a time: size
groups and diagonal tiles that end at every edge of a step's two halves, queues
that fill inside either half, thresholds that keep every pair and hardly any."""
import numpy as np
import pytest

import oracle
import paper_1711_07295_amd as ssj

pytestmark = pytest.mark.gpu

FLAGS = ssj.SSJ_FLAG_MFMA | ssj.SSJ_FLAG_SURVIVORS_ONLY


def _sets(groups, universe, seed):
    """`count` sets of `size` tokens for each (size, count); every third a copy
    of an earlier set of its size but for one token."""
    rng = np.random.default_rng(seed)
    sets = []
    for size, count in groups:
        first = len(sets)
        for i in range(count):
            s = rng.choice(universe, size, replace=False)
            if i % 3 == 2 and size > 1:
                s = sets[first + int(rng.integers(i))].copy()
                s[0] = (set(range(universe)) - set(s.tolist())).pop()
            sets.append(np.sort(s))
    off = np.concatenate([[0], np.cumsum([len(s) for s in sets])]).astype(np.uint64)
    return off, np.concatenate(sets).astype(np.uint32)


# 20 and 34 tokens: groups under and over the size from which a step covers
# several sizes; at 1/2 nearly every pair of 60 tokens survives 64 bits, at 9/10
# hardly one does
@pytest.mark.parametrize("cols", [1, 31, 32, 33, 63, 64, 65, 96, 127, 129])
@pytest.mark.parametrize("rows", [1, 33, 191, 193])
@pytest.mark.parametrize("sim,p,q", [(ssj.SSJ_SIM_JACCARD, 1, 2), (ssj.SSJ_SIM_JACCARD, 9, 10),
                                     (ssj.SSJ_SIM_COSINE, 7, 10)])
def test_groups_end_in_either_half(sim, p, q, rows, cols):
    off, tok = _sets([(20, cols), (21, 5), (34, cols), (35, 70), (36, cols), (60, rows)], 300,
                     1000 * rows + cols)
    d = ssj.to_device(off, tok)
    bm = oracle.bitmaps(off, tok, 64, oracle.BM_XOR)
    cnt, band, want = oracle.survivors(off, bm, 64, p, q, listing=True, sim=sim)
    for cap in (0, 4096):
        got, st = ssj.ssj_self_join(d, p, q, b_bits=64, sim=sim, queue_capacity=cap, flags=FLAGS)
        assert st["survivors"] == cnt and st["band_pairs"] == band
        assert np.array_equal(got, want)


@pytest.mark.parametrize("cap", [0, 4096])
@pytest.mark.parametrize("p,q", [(1, 2), (4, 5)])
def test_rows_against_other_columns(p, q, cap):
    r, s = _sets([(24, 65), (40, 193)], 200, 1), _sets([(24, 33), (32, 64), (40, 129)], 200, 2)
    got, _ = ssj.ssj_rs_join(ssj.to_device(*r), ssj.to_device(*s), p, q, b_bits=64,
                             queue_capacity=cap, flags=ssj.SSJ_FLAG_MFMA)
    assert np.array_equal(got, oracle.rs_join(*r, *s, p, q))

"""The 64-bit filter's steps of 64 columns, scored two columns at a time: size
groups and diagonal tiles that end at every edge of a step's two halves, queues
that fill inside either half, thresholds that keep every pair and hardly any."""
import numpy as np
import pytest
import torch

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


# The two columns of an accumulator are exact only if the matrix cores lose nothing of a sum
# of +-1/2 and +-2^15 onto 1.5 2^23 on its way, which no range of the result shows: every
# combination of two dot products, at a threshold on either side of each.
@pytest.mark.parametrize("place", ["low", "high", "any"])
def test_every_pair_of_dot_products(place):
    rng = np.random.default_rng({"low": 1, "high": 2, "any": 3}[place])

    def of_weight(k):
        bits = {"low": np.arange(k), "high": 63 - np.arange(k),
                "any": rng.permutation(64)[:k]}[place]
        return np.bitwise_or.reduce(np.uint64(1) << bits.astype(np.uint64), initial=np.uint64(0))

    # columns j and j + 32 of a step: weights (u, v), all 65 x 65 of them
    pairs = [(u, v) for u in range(65) for v in range(65)]
    pairs += pairs[:-len(pairs) % 32]
    cols = np.array([of_weight(w) for k in range(0, len(pairs), 32)
                     for half in (0, 1) for w in [p[half] for p in pairs[k:k + 32]]], np.uint64)
    # rows: all clear and all set (the dot products themselves), then any
    rows = np.array([0, 2**64 - 1] + list(rng.integers(0, 2**64, 46, dtype=np.uint64)), np.uint64)
    rows = np.concatenate([rows, rows])
    sizes = np.repeat([64, 65], len(rows) // 2)

    def device(n_tokens):
        off = np.concatenate([[0], np.cumsum(n_tokens)]).astype(np.uint64)
        return ssj.to_device(off, np.concatenate([np.arange(n) for n in n_tokens]))

    def bitmaps(x):
        return torch.from_numpy(x.view(np.int64).reshape(-1, 1)).cuda()

    r, s = device(sizes), device([64] * len(cols))
    rb, sb = bitmaps(rows), bitmaps(cols)
    x = rows[:, None] ^ cols[None, :]
    far = np.unpackbits(x.view(np.uint8).reshape(*x.shape, 8), axis=2).sum(2, dtype=np.int64)
    seen = set()
    for o in range(32, 65):  # kept: UB >= o, differing bits at most |r| + |s| - 2 o
        slack = sizes + 64 - 2 * o
        seen |= set(slack.tolist())
        want = np.argwhere(far <= slack[:, None]).astype(np.uint32)
        got, st = ssj.ssj_rs_join(r, s, o, 1, b_bits=64, r_bitmaps=rb, s_bitmaps=sb,
                                  sim=ssj.SSJ_SIM_OVERLAP, tile_cols=512, flags=FLAGS)
        assert st["survivors"] == len(want)
        assert np.array_equal(got.reshape(-1, 2), want)
    assert seen == set(range(0, 66))

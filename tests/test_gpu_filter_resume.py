"""Rounds that fill the survivor queue: every tile that a wave could not finish or start is
recorded once and resumed, however many of them a wave holds, at a cost that does not
grow with their number."""
import numpy as np
import pytest

import gen
import oracle
import paper_1711_07295_amd as ssj

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tiles():
    """2,880 sets of 40 tokens and 512 of 90: in tiles of one column a launch of 65,205, close to
    the most that get a wave each, so that a wave of the 1024-bit kernel (1,024 of
    them are resident) holds up to 64 resume entries."""
    rng = np.random.default_rng(5)
    sets = [np.sort(rng.choice(3 * n // 2, n, replace=False)) for n in [40] * 2880 + [90] * 512]
    off = np.concatenate([[0], np.cumsum([len(s) for s in sets])]).astype(np.uint64)
    tok = np.concatenate(sets).astype(np.uint32)
    bm = oracle.bitmaps(off, tok, 1024, oracle.BM_XOR)
    cnt, _, want = oracle.survivors(off, bm, 1024, 1, 2, listing=True)
    return ssj.to_device(off, tok), cnt, want


@pytest.mark.parametrize("flags", [ssj.SSJ_FLAG_MFMA, ssj.SSJ_FLAG_VALU])
@pytest.mark.parametrize("cap", [40_000, 700_000])
def test_waves_with_many_entries_left(tiles, cap, flags):
    d, cnt, want = tiles
    assert cnt > 2 * 700_000
    got, st = ssj.ssj_self_join(d, 1, 2, b_bits=1024, tile_cols=1, queue_capacity=cap,
                                flags=flags | ssj.SSJ_FLAG_SURVIVORS_ONLY)
    assert 63 * 1024 < st["class_tiles"][0] <= 65536 and st["filter_launches"] > cnt // cap
    assert st["survivors"] == cnt and np.array_equal(got, want)


def test_a_round_over_many_tiles_is_short():
    """25,000 tiles over a 40,000-slot queue: 0.1 ms a round (0.6 with an atomic a tile)."""
    c = gen.generate(n_sets=40_000, universe=40_000, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL,
                     size_a=30.0, size_b=0.8, size_lo=2, size_hi=500, planted_frac=0.05, seed=3)
    d = ssj.to_device(c.offsets, c.tokens)
    rounds = []
    for _ in range(2):
        _, st = ssj.ssj_self_join(d, 1, 2, b_bits=64, queue_capacity=40_000)
        assert st["class_tiles"][0] > 20_000 and st["filter_launches"] > 100
        rounds.append(st["ms_filter"] / st["filter_launches"])
    assert min(rounds) < 0.4, rounds

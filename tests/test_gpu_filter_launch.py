"""How the filter's tiles are handed out and its survivors queued: launches of
one wave per tile and persistent ones, queues of one stripe and of several,
drained once or over many rounds that resume inside tiles."""
import numpy as np
import pytest

import gen
import oracle
import paper_1711_07295_amd as ssj

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dense():
    """9,000 sets whose 64-bit bitmaps keep over 40,000 pairs at 1/2."""
    c = gen.generate(n_sets=9000, universe=500, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL,
                     size_a=20.0, size_b=0.8, size_lo=1, size_hi=60, planted_frac=0.3, seed=77)
    want = oracle.self_join(c.offsets, c.tokens, 1, 2)
    bm = oracle.bitmaps(c.offsets, c.tokens, 64, oracle.BM_XOR)
    survivors = oracle.survivors(c.offsets, bm, 64, 1, 2)[0]
    assert survivors > 40_000
    return c, ssj.to_device(c.offsets, c.tokens), want, survivors


# tile_cols 1 cuts the plan into more tiles than a launch of one wave per
# tile takes (persistent waves), 64 and the default into fewer; 40,000 slots
# make two queue stripes, 2^23 (the default) 64
@pytest.mark.parametrize("flags", [ssj.SSJ_FLAG_MFMA, ssj.SSJ_FLAG_VALU])
@pytest.mark.parametrize("tile_cols", [1, 64, 0])
@pytest.mark.parametrize("cap", [4096, 40_000, 0])
def test_tiles_and_stripes(dense, cap, tile_cols, flags):
    c, d, want, survivors = dense
    got, st = ssj.ssj_self_join(d, 1, 2, b_bits=64, queue_capacity=cap, tile_cols=tile_cols,
                                flags=flags)
    assert (st["class_tiles"][0] > 65536) == (tile_cols == 1)
    assert np.array_equal(got, want) and st["survivors"] == survivors
    assert (st["filter_launches"] > 1) == (0 < cap < survivors)


def test_later_classes_resume_from_their_tile_starts():
    """Width classes after the one that fills the queue have started none of
    their tiles; the resumed rounds run each of them once."""
    cols = [gen.generate(n_sets=n, universe=2000, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL,
                         size_a=m, size_b=0.6, size_lo=2, size_hi=600, planted_frac=0.3, seed=s)
            for n, m, s in ((8000, 8.0, 78), (3000, 150.0, 79))]
    devs = [ssj.to_device(c.offsets, c.tokens) for c in cols]
    p, q = [4, 1], [5, 2]
    one, s1 = ssj.ssj_self_join_batch(devs, p, q)
    got, st = ssj.ssj_self_join_batch(devs, p, q, queue_capacity=4096)
    assert st["n_classes"] == s1["n_classes"] >= 2
    assert st["filter_launches"] > s1["filter_launches"]
    assert st["survivors"] == s1["survivors"] > 4096
    for c, a, b, x, y in zip(cols, one, got, p, q):
        want = oracle.self_join(c.offsets, c.tokens, x, y)
        assert np.array_equal(a, want) and np.array_equal(b, want)


@pytest.fixture(scope="module")
def sparse():
    """600 sets of 33 .. 1,500 tokens: hardly two of one size, so that nearly every
    step of the filter covers columns of several sizes."""
    c = gen.generate(n_sets=600, universe=6000, zipf_s=0.8, size_dist=gen.SIZE_UNIFORM,
                     size_lo=33, size_hi=1500, planted_frac=0.5, seed=80)
    return c, ssj.to_device(c.offsets, c.tokens)


# 64 bits saturate (thresholds below every dot product: whole steps survive),
# 512 keep few; a 4,096-slot queue resumes inside such steps
@pytest.mark.parametrize("flags", [ssj.SSJ_FLAG_MFMA, ssj.SSJ_FLAG_VALU])
@pytest.mark.parametrize("b", [64, 128, 256, 512, 1024])
@pytest.mark.parametrize("sim,p,q", [(ssj.SSJ_SIM_JACCARD, 1, 2), (ssj.SSJ_SIM_JACCARD, 9, 10),
                                     (ssj.SSJ_SIM_DICE, 2, 3), (ssj.SSJ_SIM_COSINE, 3, 5),
                                     (ssj.SSJ_SIM_COSINE, 65537, 70001),
                                     (ssj.SSJ_SIM_OVERLAP, 200, 1)])
def test_steps_of_several_sizes(sparse, sim, p, q, b, flags):
    c, d = sparse
    bm = oracle.bitmaps(c.offsets, c.tokens, b, oracle.BM_XOR)
    cnt, band, want = oracle.survivors(c.offsets, bm, b, p, q, listing=True, sim=sim)
    for cap in (0, 4096):
        got, st = ssj.ssj_self_join(d, p, q, b_bits=b, sim=sim, queue_capacity=cap,
                                    flags=flags | ssj.SSJ_FLAG_SURVIVORS_ONLY)
        assert st["survivors"] == cnt and st["band_pairs"] == band
        assert np.array_equal(got, want)


@pytest.mark.parametrize("n,b,least", [(60_000, 2048, 20_000), (60_000, 4096, 20_000),
                                       (200_000, 64, 20_000), (200_000, 192, 40_000)])
def test_vector_alu_classes_are_cut_into_enough_tiles(n, b, least):
    c = gen.generate(n_sets=n, universe=n, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL, size_a=20.0,
                     size_b=0.8, size_lo=2, size_hi=500, planted_frac=0.05, seed=81)
    d = ssj.to_device(c.offsets, c.tokens)
    got, st = ssj.ssj_self_join(d, 4, 5, b_bits=b, flags=ssj.SSJ_FLAG_VALU)
    want, _ = ssj.ssj_self_join(d, 4, 5, b_bits=256, flags=ssj.SSJ_FLAG_MFMA)
    assert st["class_tiles"][0] > least and np.array_equal(got, want)


@pytest.fixture(scope="module")
def even():
    """5,000 sets of 20 .. 24 tokens: at 1/3 every pair is in the band, and many survive."""
    c = gen.generate(n_sets=5000, universe=50, zipf_s=0.5, size_dist=gen.SIZE_UNIFORM, size_lo=20,
                     size_hi=24, planted_frac=0.2, seed=82)
    return c, ssj.to_device(c.offsets, c.tokens)


# in tiles of one column every width has more tiles than get a wave each
@pytest.mark.parametrize("flags", [ssj.SSJ_FLAG_MFMA, ssj.SSJ_FLAG_VALU])
@pytest.mark.parametrize("b", [128, 256, 512, 1024])
def test_cursors_at_every_width(even, b, flags):
    c, d = even
    bm = oracle.bitmaps(c.offsets, c.tokens, b, oracle.BM_XOR)
    cnt, _, want = oracle.survivors(c.offsets, bm, b, 1, 3, listing=True)
    for cap in (0, 40_000):
        got, st = ssj.ssj_self_join(d, 1, 3, b_bits=b, tile_cols=1, queue_capacity=cap,
                                    flags=flags | ssj.SSJ_FLAG_SURVIVORS_ONLY)
        assert st["class_tiles"][0] > 65536 and (cap == 0 or st["filter_launches"] > 1)
        assert st["survivors"] == cnt > 100_000 and np.array_equal(got, want)


def test_large_wide_class_takes_the_cursors():
    """20,000 sets of one size at 2048 bits: fewer tiles than get a wave each, but more than
    0.7 ms of work; a queue that fills."""
    c = gen.generate(n_sets=20_000, universe=400, zipf_s=0.5, size_dist=gen.SIZE_UNIFORM,
                     size_lo=40, size_hi=40, planted_frac=0.3, seed=83)
    d = ssj.to_device(c.offsets, c.tokens)
    want = oracle.self_join(c.offsets, c.tokens, 4, 5)
    for cap in (0, 4096):
        got, st = ssj.ssj_self_join(d, 4, 5, b_bits=2048, queue_capacity=cap)
        assert st["class_tiles"][0] <= 65536 and (st["filter_launches"] > 1) == (cap > 0)
        assert st["survivors"] > 4096 and np.array_equal(got, want)


# the cursors' class first or last, one wave per tile in the others
@pytest.mark.parametrize("short,long", [(14_000, 1500), (2000, 9000)])
def test_full_queue_over_cursors_and_single_tiles(short, long):
    cols = [gen.generate(n_sets=n, universe=2000, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL,
                         size_a=m, size_b=0.4, size_lo=2, size_hi=600, planted_frac=0.3, seed=s)
            for n, m, s in ((short, 8.0, 84), (long, 150.0, 85))]
    devs = [ssj.to_device(c.offsets, c.tokens) for c in cols]
    p, q = [4, 1], [5, 2]
    got, st = ssj.ssj_self_join_batch(devs, p, q, tile_cols=1, queue_capacity=4096)
    tiles = st["class_tiles"][:st["n_classes"]]
    assert max(tiles) > 65536 and min(tiles) <= 65536 and st["filter_launches"] > len(tiles)
    for c, a, x, y in zip(cols, got, p, q):
        assert np.array_equal(a, oracle.self_join(c.offsets, c.tokens, x, y))

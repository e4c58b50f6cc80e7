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
    """6,000 sets whose 64-bit bitmaps keep over 50,000 pairs at 1/2."""
    c = gen.generate(n_sets=6000, universe=500, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL,
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
    assert (st["class_tiles"][0] > 16384) == (tile_cols == 1)
    assert np.array_equal(got, want) and st["survivors"] == survivors
    assert (st["filter_launches"] > 1) == (0 < cap < survivors)


def test_several_classes_resume_from_their_tile_starts():
    """Width classes after the one that fills the queue have started none of
    their tiles; the resumed rounds run each of them once."""
    c = gen.generate(n_sets=30_000, universe=3000, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL,
                     size_a=30.0, size_b=0.9, size_lo=2, size_hi=600, planted_frac=0.3, seed=78)
    d = ssj.to_device(c.offsets, c.tokens)
    one, s1 = ssj.ssj_self_join(d, 7, 10, b_bits=0)
    got, st = ssj.ssj_self_join(d, 7, 10, b_bits=0, queue_capacity=4096)
    assert st["n_classes"] == s1["n_classes"] >= 2
    assert st["filter_launches"] > s1["filter_launches"]
    assert np.array_equal(got, one) and st["survivors"] == s1["survivors"]
    assert np.array_equal(one, oracle.self_join_banded(c.offsets, c.tokens, 7, 10)[0])

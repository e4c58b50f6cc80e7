"""Verification where most survivors are reported: the lists that its waves stage fill many
times."""
import numpy as np
import pytest

import gen
import oracle
import paper_1711_07295_amd as ssj

pytestmark = pytest.mark.gpu


def _sets(n, median, seed):
    c = gen.generate(n_sets=n, universe=n, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL, size_a=median,
                     size_b=0.8, size_lo=2, size_hi=500, planted_frac=0.05, seed=seed)
    return c, ssj.to_device(c.offsets, c.tokens)


def test_survivors_are_reported_at_the_queue_s_rate():
    """Over 100 million of them: 0.03 ns each (0.09 with lists of 128 a wave)."""
    c, d = _sets(40_000, 30.0, 3)
    rates = []
    for _ in range(3):
        got, st = ssj.ssj_self_join(d, 1, 2, b_bits=64, flags=ssj.SSJ_FLAG_SURVIVORS_ONLY)
        assert len(got) == st["survivors"] > 90_000_000
        rates.append(1e6 * st["ms_verify"] / st["survivors"])
    assert min(rates) < 0.06, rates


# Overlap at 3 and 12 tokens: nearly every pair, and pairs of long sets, are results
@pytest.mark.parametrize("b", [0, 256])
@pytest.mark.parametrize("o,median", [(3, 20.0), (12, 90.0)])
def test_dense_results_match_the_oracle(o, median, b):
    c, d = _sets(2500, median, 4)
    got, st = ssj.ssj_self_join(d, o, 1, b_bits=b, sim=ssj.SSJ_SIM_OVERLAP)
    want = oracle.self_join(c.offsets, c.tokens, o, 1, sim=oracle.OVERLAP)
    assert len(want) > 300_000 and np.array_equal(got, want)


def test_overlap_pairs_of_long_sets_leave_their_merge_early():
    """20 common tokens of sets of about 200: 0.45 ns a survivor (0.73 with every token merged)."""
    c = gen.generate(n_sets=20_011, universe=20_011, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL,
                     size_a=150.0, size_b=0.8, size_lo=2, size_hi=2000, planted_frac=0.05, seed=4)
    d = ssj.to_device(c.offsets, c.tokens)
    rates = []
    for _ in range(3):
        _, st = ssj.ssj_self_join(d, 20, 1, b_bits=0, sim=ssj.SSJ_SIM_OVERLAP)
        assert st["survivors"] > 100_000_000
        rates.append(1e6 * st["ms_verify"] / st["survivors"])
    assert min(rates) < 0.58, rates

"""The one-launch preparation of small spaces and the one-launch end of calls
with few results, at the sizes where the general kernels take over."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_1711_07295_amd as ssj

pytestmark = pytest.mark.gpu


def _dev(c):
    return ssj.to_device(c.offsets, c.tokens)


@pytest.mark.parametrize("b", [0, 64])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025, 8191, 8192, 8193])
def test_set_counts(n, b):
    c = gen.generate(n_sets=n, universe=max(64, n), zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL,
                     size_a=9.0, size_b=0.7, size_lo=1, size_hi=300, planted_frac=0.3, seed=90 + n)
    got, st = ssj.ssj_self_join(_dev(c), 7, 10, b_bits=b)
    want, band = oracle.self_join_banded(c.offsets, c.tokens, 7, 10)
    assert np.array_equal(got, want) and st["band_pairs"] == band


@pytest.mark.parametrize("extra", [0, 1, 2, 95])
def test_result_counts(extra):
    """91 identical sets give 4,095 pairs; `extra` pairs of their own more."""
    sets = [list(range(10, 17))] * 91
    for k in range(extra):
        sets += [[1000 + 10 * k + x for x in range(5)]] * 2
    rng = np.random.default_rng(extra)
    c = gen.from_lists([sets[k] for k in rng.permutation(len(sets))])
    got, st = ssj.ssj_self_join(_dev(c), 9, 10)
    assert st["results"] == 4095 + extra
    assert np.array_equal(got, oracle.self_join(c.offsets, c.tokens, 9, 10))


@pytest.mark.parametrize("step", [1, 2, 256])
def test_keys_that_share_their_digits(step):
    """8,192 sets of one size, so that all have one sort key; 64 (32) equal ones, `step` apart, whose
    pairs share none, half or all of the two low digits of their result keys."""
    rng = np.random.default_rng(step)
    sets = [np.sort(rng.choice(4000, 8, replace=False)) for _ in range(8192)]
    for k in range(64):
        sets[k * step if step < 256 else k % 32 * step] = np.arange(5000, 5008)
    c = gen.from_lists(sets)
    got, _ = ssj.ssj_self_join(_dev(c), 9, 10)
    want = oracle.self_join(c.offsets, c.tokens, 9, 10)
    assert len(want) >= (2016 if step < 256 else 496) and np.array_equal(got, want)


@pytest.mark.parametrize("n_sides", [1, 2, 1024, 1025])
def test_side_counts(n_sides):
    """Many sides, empty ones and empty sets among them."""
    rng = np.random.default_rng(n_sides)
    cols = []
    for k in range(n_sides):
        n = int(rng.integers(0, 8))
        cols.append(gen.from_lists([np.unique(rng.integers(0, 12, int(rng.integers(0, 9))))
                                    for _ in range(n)]))
    got, _ = ssj.ssj_self_join_batch([_dev(c) for c in cols], [1] * n_sides, [2] * n_sides)
    for c, g in zip(cols, got):
        assert np.array_equal(g, oracle.self_join(c.offsets, c.tokens, 1, 2))


def test_long_side_of_few_sets():
    """Few sets whose token counts pass the bound of the one-launch preparation."""
    rng = np.random.default_rng(5)
    base = np.unique(rng.integers(0, 400_000, 90_000))
    sets = [base, base[:-7], np.unique(rng.integers(0, 400_000, 60_000)), base[3:100]]
    c = gen.from_lists(sets)
    got, _ = ssj.ssj_self_join(_dev(c), 4, 5, b_bits=0)
    assert np.array_equal(got, oracle.self_join(c.offsets, c.tokens, 4, 5))


def test_bad_offsets_leave_the_small_path_with_their_error():
    c = gen.generate(n_sets=500, universe=500, zipf_s=1.0, size_lo=2, size_hi=40, seed=91)
    for k, v in ((0, 1), (250, int(c.offsets[-1]) + 1), (250, 0), (500, int(c.offsets[-1]) - 1)):
        off = c.offsets.copy()
        off[k] = v
        for b in (0, 64, 2048):
            with pytest.raises(ssj.SsjError) as e:
                ssj.ssj_self_join(ssj.to_device(off, c.tokens), 4, 5, b_bits=b)
            assert e.value.status == ssj.SSJ_E_INVALID


def test_rs_join_reports_the_first_collection_s_error():
    """R malformed, S with a set larger than is handled: invalid, whether R is prepared in one
    launch or not; S alone: unsupported."""
    n = 1 << 25
    big = ssj.DeviceSets(torch.tensor([0, n], dtype=torch.int64, device="cuda"),
                         torch.arange(n, dtype=torch.int32, device="cuda"))
    for k, status in ((100, ssj.SSJ_E_INVALID), (9000, ssj.SSJ_E_INVALID),
                      (0, ssj.SSJ_E_UNSUPPORTED)):
        off = np.arange(max(k, 5) + 1, dtype=np.uint64)
        if k:
            off[k // 2] = 1 << 40
        r = ssj.to_device(off, np.zeros(max(k, 5), dtype=np.uint32))
        with pytest.raises(ssj.SsjError) as e:
            ssj.ssj_rs_join(r, big, 4, 5)
        assert e.value.status == status

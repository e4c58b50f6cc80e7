"""Bitmap-Next with every token probing on its own: long probe chains, wraps and
saturation at the widths of the segmented and of the wave-per-set build; and
the checks of the offsets that the build makes on its way."""
import time

import numpy as np
import pytest
import torch

import gen
import oracle
import paper_1711_07295_amd as ssj

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [64, 128, 192, 448, 512, 640, 1024, 2048, 4096])
def test_next_probe_chains(b):
    rng = np.random.default_rng(b)
    sets = []
    for n in (0, 1, 2, b // 2, b - 1, b, b + 1):
        sets.append(np.arange(n) * b + b - 1)          # one residue: one chain, wrapping
        sets.append(np.arange(n) * b + 31)             # ... across words
        sets.append(np.arange(n) + 5 * b - 3)          # consecutive residues
        sets.append(np.sort(rng.choice(40 * b, n, replace=False)))
        sets.append(np.sort(rng.choice(8, n) + b * np.arange(n)))  # eight residues
    sets = [sets[k] for k in rng.permutation(len(sets))] * 9  # over a segment of 256 sets
    c = gen.from_lists(sets)
    got = ssj.ssj_build_bitmaps(ssj.to_device(c.offsets, c.tokens), b, ssj.SSJ_BM_NEXT)
    want = oracle.bitmaps(c.offsets, c.tokens, b, oracle.BM_NEXT)
    assert np.array_equal(got.cpu().numpy().view(np.uint64), want)


@pytest.mark.parametrize("b", [64, 1024, 4096])
@pytest.mark.parametrize("method", [ssj.SSJ_BM_XOR, ssj.SSJ_BM_NEXT])
def test_malformed_offsets_wherever_they_are(method, b):
    c = gen.generate(n_sets=700, universe=900, zipf_s=1.0, size_lo=1, size_hi=30, seed=92)
    last = int(c.offsets[-1])
    for k, v in ((0, 1), (1, last + 1), (255, 0), (256, last + 5), (257, 2), (699, last + 1),
                 (700, last - 1), (700, last + 1), (300, 1 << 40)):
        off = c.offsets.copy()
        off[k] = v
        with pytest.raises(ssj.SsjError) as e:
            ssj.ssj_build_bitmaps(ssj.to_device(off, c.tokens), b, method)
        assert e.value.status == ssj.SSJ_E_INVALID, (k, v)
    off = c.offsets.copy()
    tok = c.tokens.copy()
    k = int(np.flatnonzero(np.diff(off.astype(np.int64)) > 1)[200])
    tok[int(off[k]) + 1] = tok[int(off[k])]
    with pytest.raises(ssj.SsjError) as e:
        ssj.ssj_build_bitmaps(ssj.to_device(off, tok), b, method)
    assert e.value.status == ssj.SSJ_E_UNSORTED


# a wave per set up to 65,536 sets, segments of 256 sets from there on
@pytest.mark.parametrize("n", [65_536, 65_537])
@pytest.mark.parametrize("b", [64, 192, 512, 1024, 2048])
def test_next_by_sets_and_by_segments(b, n):
    rng = np.random.default_rng(b)
    chains = []
    for k in (1, b // 2, b - 1, b, b + 1):
        chains.append(np.arange(k) * b + b - 1)
        chains.append(np.sort(rng.choice(8, k) + b * np.arange(k)))
    sets = [chains[k % 10] if k % 500 < 10 else np.array([7 * k % 1000]) for k in range(n)]
    c = gen.from_lists(sets)
    got = ssj.ssj_build_bitmaps(ssj.to_device(c.offsets, c.tokens), b, ssj.SSJ_BM_NEXT)
    want = oracle.bitmaps(c.offsets, c.tokens, b, oracle.BM_NEXT)
    assert np.array_equal(got.cpu().numpy().view(np.uint64), want)


def test_next_of_few_large_sets_uses_the_whole_gpu():
    """4,000 sets of about 550 tokens at 64 bits: 0.03 ms (0.25 with a workgroup per 256)."""
    c = gen.generate(n_sets=4000, universe=20_000, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL,
                     size_a=400.0, size_b=0.8, size_lo=2, size_hi=4000, planted_frac=0.05, seed=12)
    d = ssj.to_device(c.offsets, c.tokens)
    best = 1.0
    for _ in range(20):
        torch.cuda.synchronize()
        t = time.perf_counter()
        ssj.ssj_build_bitmaps(d, 64, ssj.SSJ_BM_NEXT)
        best = min(best, time.perf_counter() - t)
    assert best < 0.12e-3

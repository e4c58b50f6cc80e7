"""Bitmap-Next with every token probing on its own: long probe chains, wraps and
saturation at the widths of the segmented and of the wave-per-set build; and
the checks of the offsets that the build makes on its way."""
import numpy as np
import pytest

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

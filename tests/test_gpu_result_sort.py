"""The order of result lists of every size class of the sort, and the size tables
of sides whose sets skip most sizes."""
import numpy as np
import pytest

import oracle
import paper_1711_07295_amd as ssj

pytestmark = pytest.mark.gpu


# r x s equal sets: exactly that many results, around a sort block (2,048 keys),
# the shortest sorted list (4,097), 64 and 160 blocks
@pytest.mark.parametrize("r,s", [(1, 4097), (2, 2049), (128, 16), (17, 361), (256, 512),
                                 (241, 544), (511, 640), (512, 640), (577, 568), (700, 700)])
def test_results_are_in_order(r, s):
    def side(n, every):
        # the equal sets are every `every`-th; the others pair with nothing
        total = n * every
        tok = np.arange(4 * total, dtype=np.uint32).reshape(total, 4) + 1000 * every
        tok[::every] = [1, 2, 3, 4]
        return np.arange(total + 1, dtype=np.uint64) * 4, tok.reshape(-1)

    (ro, rt), (so, st) = side(r, 3), side(s, 2)
    st = np.where(st > 4, st + 10_000_000, st).astype(np.uint32)
    got, _ = ssj.ssj_rs_join(ssj.to_device(ro, rt), ssj.to_device(so, st), 4, 5)
    want = np.stack(np.meshgrid(np.arange(r) * 3, np.arange(s) * 2, indexing="ij"), -1)
    assert len(got) == r * s and np.array_equal(got, want.reshape(-1, 2).astype(got.dtype))


# sides of 1 .. 130 sets whose sizes leave gaps of 0, 3, 4, 5, 63, 64, 65 and 1,500
# sizes below, between and above them
@pytest.mark.parametrize("sizes", [(1,), (1, 2, 3), (1, 5, 9, 10), (4, 5, 70, 134, 199),
                                   (1500,), (2, 1500, 1500), tuple(range(3, 133))])
def test_batch_sides_that_skip_sizes(sizes):
    rng = np.random.default_rng(len(sizes))
    n = 8200  # more sets than one launch prepares
    many = rng.integers(3, 9, n)
    many[-1] = 1600

    def make(sz):
        off = np.concatenate([[0], np.cumsum(sz)]).astype(np.uint64)
        tok = np.concatenate([np.sort(rng.choice(1800, z, replace=False)) for z in sz])
        return off, tok.astype(np.uint32)

    insts = [make(many), make(sizes), make(tuple(sizes) * 2)]
    got, _ = ssj.ssj_self_join_batch([ssj.to_device(o, t) for o, t in insts], [1, 1, 1], [2, 2, 2])
    for (o, t), g in zip(insts, got):
        assert np.array_equal(g, oracle.self_join(o, t, 1, 2))

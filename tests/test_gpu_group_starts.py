"""The size tables of sides whose sets skip most sizes."""
import numpy as np
import pytest

import oracle
import paper_1711_07295_amd as ssj

pytestmark = pytest.mark.gpu


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

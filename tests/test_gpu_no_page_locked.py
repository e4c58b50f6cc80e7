"""Calls in a process that gets no page-locked memory (a container's limit on locked pages):
every form of call returns what it returns elsewhere.  A small library loaded first answers
the allocation for them, as an allocator without memory would."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <stddef.h>
int asked = 0;
/* hipErrorOutOfMemory */
int hipHostMalloc(void **p, size_t n, unsigned flags) { (void)n; (void)flags; *p = NULL; ++asked; return 2; }
"""

CALLS = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
import gen, oracle
import paper_1711_07295_amd as ssj

def sets(n, seed, median=15.0):
    c = gen.generate(n_sets=n, universe=3000, zipf_s=1.0, size_dist=gen.SIZE_LOGNORMAL,
                     size_a=median, size_b=0.8, size_lo=1, size_hi=300, planted_frac=0.3, seed=seed)
    return c, ssj.to_device(c.offsets, c.tokens)

for n in (600, 20_000):  # one-launch and general preparation; few results and many
    c, d = sets(n, n)
    want = oracle.self_join(c.offsets, c.tokens, 7, 10)
    for b in (0, 64):
        assert np.array_equal(ssj.ssj_self_join(d, 7, 10, b_bits=b)[0], want)
    assert np.array_equal(ssj.ssj_self_join(d, 7, 10, b_bits=64, queue_capacity=4096)[0], want)
    assert np.array_equal(ssj.ssj_self_join(d, 7, 10, b_bits=64, flags=ssj.SSJ_FLAG_CUTOFF)[0], want)
    for got in ssj.ssj_self_join_batch([d, d], [7, 7], [10, 10])[0]:
        assert np.array_equal(got, want)
    with ssj.Plan([d], [7], [10]) as plan:
        for _ in range(2):
            assert np.array_equal(plan.execute()[0][0], want)
    q, dq = sets(50, 3)
    with ssj.Index(d) as idx:
        got = idx.query([dq], [7], [10])[0][0]
    assert np.array_equal(got, oracle.rs_join(q.offsets, q.tokens, c.offsets, c.tokens, 7, 10))
    bm = ssj.ssj_build_bitmaps(d, 128).cpu().numpy().view(np.uint64)
    assert np.array_equal(bm, oracle.bitmaps(c.offsets, c.tokens, 128, oracle.BM_XOR))
assert ctypes.c_int.in_dll(shim, "asked").value > 0
print("same results")
"""


def test_every_call_works_without_page_locked_memory(tmp_path):
    src, lib = tmp_path / "shim.c", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", str(src), "-o", str(lib)], check=True)
    env = dict(os.environ, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", CALLS, str(lib)], capture_output=True, text=True,
                       timeout=100, cwd=ROOT, env=env)
    assert r.returncode == 0 and "same results" in r.stdout, r.stderr[-2000:]

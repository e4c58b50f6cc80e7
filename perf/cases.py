"""Performance cases of the library: what its users call, over the sizes they call it with.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges, ``prepare`` makes a case's
input on the GPU from a seed, ``run`` makes one call through the public entry points, ``work`` counts
the bytes and operations no method can do without, and ``exact`` recomputes the outputs with plain torch
where that is quick.

Inputs have the structure of the paper's collections (and of the repository's named workloads):
Zipf-like tokens numbered by ascending frequency, log-normal or uniform set sizes, some sets near
duplicates of others.  A case's ``spread`` draws which sets there are; the seed of an input then
shuffles their order and renumbers tokens of about one frequency, so that bitmaps, survivors and
pairs are others with every seed while the number of similar pairs stays the case's own.
"""
import math
import random

import numpy as np
import torch

import paper_1711_07295_amd as ssj

DEVICE = "cuda"
SIM = {"jaccard": ssj.SSJ_SIM_JACCARD, "dice": ssj.SSJ_SIM_DICE, "cosine": ssj.SSJ_SIM_COSINE}
METHOD = {"xor": ssj.SSJ_BM_XOR, "set": ssj.SSJ_BM_SET, "next": ssj.SSJ_BM_NEXT}
THRESHOLDS = [(1, 2), (7, 10), (4, 5), (9, 10), (19, 20)]


def listed():
    """b is the bitmap width (0: the library's automatic widths per size class); sizes are log-normal
    with the given median and sigma, or uniform in lo..hi when sigma is 0."""
    return [
        # one small collection with the binding's defaults (64-bit bitmaps): a call's latency
        dict(name="join-1k", kind="join", spread=1, n=1000, universe=1000, zipf=1.0, median=0.0,
             sigma=0.0,
             lo=5, hi=50, planted=0.05, p=4, q=5, sim="jaccard", b=64),
        # the benchmark's workload: one million sets at 4/5, automatic widths
        dict(name="join-1m", kind="join", spread=1, n=1_000_000, universe=1_000_000, zipf=1.1,
             median=20.0,
             sigma=0.8, lo=2, hi=500, planted=0.05, p=4, q=5, sim="jaccard", b=0),
        # many short sets at a high threshold (titles, queries): near-duplicate detection
        dict(name="join-4m-short", kind="join", spread=1, n=4_000_000, universe=2_000_000, zipf=1.0,
             median=12.0, sigma=0.6, lo=2, hi=200, planted=0.02, p=19, q=20, sim="jaccard", b=0),
        # long documents at a low threshold: wide bitmaps and long merges; an odd count
        dict(name="join-long", kind="join", spread=1, n=60_013, universe=60_013, zipf=1.0, median=150.0,
             sigma=0.8, lo=2, hi=2000, planted=0.05, p=1, q=2, sim="jaccard", b=0),
        # a user with bitmaps of their own (Bitmap-Set, one width) and another similarity
        dict(name="join-given", kind="given", spread=1, n=200_003, universe=200_003, zipf=1.1,
             median=20.0,
             sigma=0.8, lo=2, hi=500, planted=0.05, p=9, q=10, sim="dice", b=256, method="set"),
        # a few thousand new records against a table: R-S join, Cosine
        dict(name="rs-3k", kind="rs", spread=1, n_r=3001, n=300_007, universe=300_007, zipf=1.1,
             median=30.0,
             sigma=0.8, lo=2, hi=500, copies=0.2, p=4, q=5, sim="cosine", b=0),
        # many uneven collections, each at its own threshold, in one call
        dict(name="batch-48", kind="batch", instances=48, spread=1, n_min=1000, n_max=200_000,
             m_min=5.0, m_max=200.0, hi=2000),
        # the same join run again and again on changing tokens: a prepared plan of six collections
        dict(name="plan-6", kind="plan", instances=6, spread=2, n_min=3000, n_max=60_000,
             m_min=8.0, m_max=60.0, hi=500),
        # one new record against a resident index: the served form's smallest call
        dict(name="query-1", kind="query", spread=1, n_r=1, n=1_000_000, universe=400_000, zipf=1.1,
             median=30.0, sigma=0.8, lo=2, hi=500, copies=0.2, p=7, q=10, sim="jaccard", b=0),
        # a large query batch against the resident collection's full size
        dict(name="query-2k", kind="query", spread=1, n_r=2003, n=5_000_000, universe=2_000_000,
             zipf=1.1,
             median=30.0, sigma=0.8, lo=2, hi=500, copies=0.2, p=7, q=10, sim="jaccard", b=0),
        # bitmaps of a collection, to keep and join with later
        dict(name="bitmaps-1m", kind="bitmaps", spread=1, n=1_000_000, universe=1_000_000, zipf=1.1,
             median=20.0, sigma=0.8, lo=2, hi=500, method="xor", b=128),
        # the same in a loop that must not allocate, with the generator of low thresholds
        dict(name="bitmaps-next-20k", kind="noalloc", spread=1, n=20_011, universe=20_011, zipf=1.1,
             median=30.0, sigma=0.8, lo=2, hi=500, method="next", b=512),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw(rng):
    kind = rng.choice(["join", "join", "join", "given", "rs", "batch", "plan", "query", "query",
                       "bitmaps", "noalloc"])
    if kind in ("batch", "plan"):
        hi = int(_log(rng, 4000, 200_000 if kind == "batch" else 60_000))
        return dict(kind=kind, instances=rng.randint(2, 48 if kind == "batch" else 8),
                    spread=rng.randrange(1 << 20), n_min=1000, n_max=hi, m_min=5.0,
                    m_max=_log(rng, 20, 200), hi=2000)
    median = round(_log(rng, 8, 150 if kind in ("join", "batch") else 40), 2)
    c = dict(kind=kind, spread=rng.randrange(1 << 20), n=0, universe=0,
             zipf=round(rng.uniform(0.9, 1.2), 3), median=median,
             sigma=round(rng.uniform(0.5, 0.8), 2), lo=2, hi=2000 if median > 60 else 500)
    if kind in ("bitmaps", "noalloc"):
        c["n"] = int(_log(rng, 500, 1_000_000))
        c["method"] = rng.choice(["xor", "xor", "set", "next"])
        c["b"] = rng.choice([64, 128, 192, 256, 512, 1024, 2048])
        if c["b"] > 256 or c["method"] == "next":
            c["n"] = min(c["n"], 200_000)
    else:
        p, q = rng.choice(THRESHOLDS if median > 25 else THRESHOLDS[1:])
        c["p"], c["q"], c["sim"] = p, q, rng.choice(["jaccard", "jaccard", "dice", "cosine"])
        if c["sim"] != "jaccard":  # the same overlap asked of two sets of one size
            c["p"], c["q"] = max([(7, 10), (4, 5), (9, 10), (19, 20)],
                                 key=lambda t: -abs(t[0] / t[1] - 2 * p / (p + q)))
        c["b"] = rng.choice([0, 0, 64, 128, 256]) if kind in ("join", "rs") else 0
        if kind == "join":
            c["n"], c["planted"] = int(_log(rng, 1000, 1_500_000 / (median / 12))), 0.05
            if c["b"] == 64 and median > 25:
                c["b"] = 128
            if c["b"] and median > 40:
                c["b"] = 512
        elif kind == "given":
            c["n"], c["planted"], c["method"] = int(_log(rng, 1000, 200_000)), 0.05, \
                rng.choice(["xor", "set", "next"])
            c["b"] = rng.choice([192, 256, 512])
        else:
            c["n"], c["copies"] = int(_log(rng, 20_000, 300_000 if kind == "rs" else 1_500_000)), 0.2
            c["n_r"] = int(_log(rng, 1, 8000))
            if c["b"] == 64:
                c["b"] = 128
    c["universe"] = max(c["n"] // (1 if kind != "query" else 2), int(50 * median))
    return c


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= most:
            return c


# ------------------------------------------------------------------------------------------ input
def _instances(case):
    """Parameters of a batch's collections (the same for every seed of its inputs)."""
    rng = random.Random(case["spread"])
    out = []
    for _ in range(case["instances"]):
        m = _log(rng, case["m_min"], case["m_max"])
        n = int(round(_log(rng, case["n_min"], case["n_max"])))
        p, q = rng.choice(THRESHOLDS[:4])
        out.append(dict(n=n, universe=max(n, int(50 * m)), zipf=rng.uniform(0.8, 1.3), median=m,
                        sigma=0.8, lo=2, hi=case["hi"], planted=0.05, p=p, q=q,
                        spread=rng.randrange(1 << 30)))
    return out


def _sizes(c, n, gen, device):
    if c["sigma"] == 0:
        return torch.randint(c["lo"], c["hi"] + 1, (n,), generator=gen, device=device)
    z = torch.randn(n, generator=gen, device=device, dtype=torch.float64)
    return torch.exp(math.log(c["median"]) + c["sigma"] * z).round().long().clamp_(c["lo"], c["hi"])


def _replaced(c):
    """Share of a copy's draws that differ from its base's: one in ten, fewer where the threshold
    asked for would never match such a copy."""
    if "p" not in c:
        return 0.1
    t = c["p"] / c["q"]
    return min(0.1, 0.6 * (1 - t) / (1 + t))


def _collection(c, n, gen, mix, copy=None, base=None, place=None):
    """n sets as (int64 offsets, int32 tokens): the first size-many distinct tokens of a run of Zipf
    draws; sets ``copy`` repeat the draws of sets ``base`` with some replaced.  ``gen`` draws the
    sets, ``mix`` their order (unless given as ``place``) and the tokens' numbers."""
    dev = DEVICE
    size = _sizes(c, n, gen, dev)
    if place is None:
        place = torch.randperm(n, generator=mix, device=dev)
    if copy is not None:
        size[copy] = size[base]
    n_draw = size + (size * 3) // 5 + 6
    end = n_draw.cumsum(0)
    start = end - n_draw
    total = int(end[-1])
    owner = torch.repeat_interleave(torch.arange(n, device=dev), n_draw, output_size=total)
    cdf = torch.arange(1, c["universe"] + 1, device=dev, dtype=torch.float64)
    cdf = cdf.pow_(-c["zipf"]).cumsum_(0)
    u = torch.rand(total, generator=gen, device=dev, dtype=torch.float64).mul_(cdf[-1])
    tok = torch.searchsorted(cdf, u).clamp_(max=c["universe"] - 1)
    del u
    if copy is not None:
        src = torch.arange(n, device=dev)
        src[copy] = base
        at = torch.arange(total, device=dev) - start[owner] + start[src[owner]]
        kept = torch.rand(total, generator=gen, device=dev) >= _replaced(c)
        tok = torch.where(kept, tok[at], tok)
        del at, kept, src
    order = torch.argsort(torch.bincount(tok, minlength=c["universe"]), stable=True)
    rename = torch.empty_like(order)
    # ascending frequency, shuffled within every 1024 tokens
    rank = torch.arange(c["universe"], device=dev)
    rank = torch.argsort(rank // 1024 + torch.rand(c["universe"], generator=mix, device=dev,
                                                   dtype=torch.float64))
    rename[order] = rank
    key, perm = torch.sort((place[owner] << 32) | rename[tok], stable=True)
    del tok
    fresh = torch.ones(total, dtype=torch.bool, device=dev)
    fresh[1:] = key[1:] != key[:-1]
    seen = torch.zeros(total, dtype=torch.bool, device=dev)
    seen[perm] = fresh
    count = seen.cumsum(0)
    before = torch.zeros(n, dtype=torch.int64, device=dev)
    before[1:] = count[end[:-1] - 1]
    keep = seen & (count - before[owner] <= size[owner])
    tokens = (key[keep[perm]] & 0xFFFFFFFF).int()
    offsets = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    offsets[1:] = torch.bincount(place[owner[keep]], minlength=n).cumsum(0)
    return offsets, tokens


def _planted(c, n, gen):
    """Sets that repeat another: ``planted`` of n, in clusters of about ten around one base each."""
    k = int(round(c.get("planted", 0.0) * n))
    if k < 2:
        return None, None
    perm = torch.randperm(n, generator=gen, device=DEVICE)
    n_base = max(1, k // 11)
    copy = perm[n_base:k]
    return copy, perm[torch.randint(0, n_base, (len(copy),), generator=gen, device=DEVICE)]


def _sets(offsets, tokens):
    return ssj.DeviceSets(offsets.contiguous(), tokens.contiguous())


def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed & 0x7FFFFFFFFFFF)
    return g


def _self_sets(c, mix):
    gen = _generator(c["spread"])
    copy, base = _planted(c, c["n"], gen)
    return _sets(*_collection(c, c["n"], gen, mix, copy, base))


def _two_sides(c, mix):
    """n resident sets and n_r others of the same distribution, ``copies`` of these near a resident
    (one at least)."""
    n, n_r = c["n"], c["n_r"]
    gen = _generator(c["spread"])
    copy = n + torch.arange(max(1, int(round(c["copies"] * n_r))), device=DEVICE)
    base = torch.randint(0, n, (len(copy),), generator=gen, device=DEVICE)
    place = torch.cat([torch.randperm(n, generator=mix, device=DEVICE),
                       n + torch.randperm(n_r, generator=mix, device=DEVICE)])
    off, tok = _collection(c, n + n_r, gen, mix, copy, base, place)
    cut = int(off[n])
    return _sets(off[n:] - cut, tok[cut:].clone()), _sets(off[:n + 1].clone(), tok[:cut].clone())


class _State(dict):
    """A case's input; a plan or an index among it is closed with it."""

    def __del__(self):
        for v in self.values():
            if isinstance(v, (ssj.Plan, ssj.Index)):
                v.close()


def prepare(case, seed):
    mix = _generator(seed)
    st, kind = _State(case=case), case["kind"]
    if kind in ("join", "given", "bitmaps", "noalloc"):
        st["s"] = _self_sets(case, mix)
        if kind == "given":
            st["bitmaps"] = ssj.ssj_build_bitmaps(st["s"], case["b"], METHOD[case["method"]])
        if kind == "noalloc":
            st["out"] = torch.empty((case["n"], case["b"] // 64), dtype=torch.int64, device=DEVICE)
    elif kind == "rs":
        st["r"], st["s"] = _two_sides(case, mix)
    elif kind == "query":
        st["r"], s = _two_sides(case, mix)
        st["index"] = ssj.Index(s)
    else:
        inst = _instances(case)
        st["sets"] = [_self_sets(c, mix) for c in inst]
        st["p"], st["q"] = [c["p"] for c in inst], [c["q"] for c in inst]
        if kind == "plan":
            st["plan"] = ssj.Plan(st["sets"], st["p"], st["q"])
    return st


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "join":
        return ssj.ssj_self_join(st["s"], c["p"], c["q"], b_bits=c["b"], sim=SIM[c["sim"]])[0]
    if kind == "given":
        return ssj.ssj_self_join(st["s"], c["p"], c["q"], b_bits=c["b"], bitmaps=st["bitmaps"],
                                 sim=SIM[c["sim"]])[0]
    if kind == "rs":
        return ssj.ssj_rs_join(st["r"], st["s"], c["p"], c["q"], b_bits=c["b"], sim=SIM[c["sim"]])[0]
    if kind == "batch":
        return ssj.ssj_self_join_batch(st["sets"], st["p"], st["q"])[0]
    if kind == "plan":
        return st["plan"].execute()[0]
    if kind == "query":
        return st["index"].query([st["r"]], [c["p"]], [c["q"]], sim=SIM[c["sim"]])[0]
    if kind == "bitmaps":
        return ssj.ssj_build_bitmaps(st["s"], c["b"], METHOD[c["method"]])
    return ssj.ssj_build_bitmaps_noalloc(st["s"], c["b"], st["out"], METHOD[c["method"]])


# ------------------------------------------------------------------------------------------- work
_SAMPLE = 4096


def _quantiles(c):
    """Set sizes at the middle of _SAMPLE equal shares of the size distribution, ascending."""
    u = (np.arange(_SAMPLE) + 0.5) / _SAMPLE
    if c["sigma"] == 0:
        return np.floor(c["lo"] + u * (c["hi"] + 1 - c["lo"]))
    z = math.sqrt(2) * torch.erfinv(torch.from_numpy(2 * u - 1)).numpy()
    return np.clip(np.round(np.exp(math.log(c["median"]) + c["sigma"] * z)), c["lo"], c["hi"])


def _band_share(c, sim):
    """Share of set pairs whose sizes alone do not rule them out (the length filter)."""
    s, t = _quantiles(c), c["p"] / c["q"]
    least = {"jaccard": t, "dice": t / (2 - t), "cosine": t * t}[sim]
    first = np.searchsorted(s, np.ceil(s * least - 1e-9), side="left")
    last = np.searchsorted(s, np.floor(s / least + 1e-9), side="right")
    return float((last - first).mean() / _SAMPLE)


def work(case):
    """Each offset and token read once, each bitmap written once; per pair of the length band one
    64-bit test (the dot product of two vectors of 64 signs). A resident index is already
    there: a query reads its narrowest bitmaps, not its tokens."""
    kind = case["kind"]
    if kind in ("batch", "plan"):
        parts = [dict(c, kind="join", sim="jaccard", b=0) for c in _instances(case)]
        done = [work(c) for c in parts]
        return {k: sum(w[k] for w in done) for k in ("bytes", "flops")}
    mean = float(_quantiles(case).mean())
    n = case["n"]
    if kind in ("bitmaps", "noalloc"):
        return {"bytes": n * (8 + 4 * mean + case["b"] / 8), "flops": n * mean}
    share = _band_share(case, case["sim"])
    if kind in ("rs", "query"):
        own = n * (8 + 4 * mean) if kind == "rs" else n * 8
        return {"bytes": own + case["n_r"] * (8 + 4 * mean), "flops": case["n_r"] * n * share * 128}
    given = case["b"] / 8 if kind == "given" else 0
    return {"bytes": n * (8 + 4 * mean + given), "flops": 0.5 * n * n * share * 128}


def _cost(case):
    """A rough time of one pass, to keep drawn cases at or below the largest listed one."""
    w = work(case)
    wide = 1 + case.get("median", case.get("m_max", 20.0)) / 30
    return w["flops"] * wide / 2.5e15 + w["bytes"] / 1e12


# ------------------------------------------------------------------------------------------ exact
def exact(case, seed):
    kind = case["kind"]
    if kind in ("bitmaps", "noalloc") and case["n"] * case["b"] <= 1 << 28:
        return _exact_bitmaps(case, prepare(case, seed)["s"])
    if kind == "join" and case["n"] <= 4000 and case["universe"] <= 20_000:
        return _exact_join(case, prepare(case, seed)["s"])
    return None


def _members(s, width, mod):
    """0/1 matrix of sets against their tokens' residues, summed (float64)."""
    off = s.offsets
    owner = torch.repeat_interleave(torch.arange(s.n_sets, device=off.device), off[1:] - off[:-1])
    m = torch.zeros(s.n_sets * width, dtype=torch.float64, device=off.device)
    m.index_add_(0, owner * width + s.tokens.long() % mod,
                 torch.ones(s.n_tokens, dtype=torch.float64, device=off.device))
    return m.view(s.n_sets, width)


def _exact_bitmaps(case, s):
    b = case["b"]
    if case["method"] == "next":
        bits = _next_bits(s, b)
    else:
        count = _members(s, b, b)
        bits = (count.long() & 1) if case["method"] == "xor" else (count > 0).long()
    shift = torch.arange(64, device=bits.device)
    return (bits.view(s.n_sets, b // 64, 64) << shift).sum(2)


def _next_bits(s, b):
    """Bitmap-Next: each token sets the first unset bit at or after its residue, cyclically; a set of
    at least b tokens sets every bit."""
    off, tok = s.offsets, s.tokens.long()
    size = off[1:] - off[:-1]
    bits = torch.zeros((s.n_sets, b), dtype=torch.int64, device=off.device)
    bits[size >= b] = 1
    for k in range(int(size.max()) if s.n_sets else 0):
        live = torch.nonzero((size > k) & (size < b)).flatten()
        at = tok[off[live] + k] % b
        while len(live):  # one probe further for those whose bit is taken
            taken = bits[live, at] == 1
            bits[live[~taken], at[~taken]] = 1
            live, at = live[taken], (at[taken] + 1) % b
    return bits


def _exact_join(case, s):
    m = _members(s, case["universe"], 1 << 32)
    size = m.sum(1)
    over = m @ m.T
    p, q, a, c = case["p"], case["q"], size[:, None], size[None, :]
    near = {"jaccard": lambda: q * over >= p * (a + c - over),
            "dice": lambda: 2 * q * over >= p * (a + c),
            "cosine": lambda: (q * over) ** 2 >= p * p * a * c}[case["sim"]]()
    near &= (a > 0) & (c > 0)
    return torch.nonzero(torch.triu(near, diagonal=1)).cpu().numpy().astype(np.uint32)

"""The GEMM planners' promises, checked on the host over random products: no
plan adds an output's terms in longer chains than the plan that it replaced, and
splits stay within the room given."""
import math
import random

from native_plan import planner  # noqa: F401  (fixture)

# BK, waves that share a slab's k, accumulators per output: the plan's tiles, and the older plan's (one accumulator)
TILES = {"HUGE": (32, 1, 2), "BIG": (64, 2, 4), "MID": (32, 1, 4), "DUO": (64, 2, 2), "SMALL": (128, 8, 1), "NARROW": (32, 2, 1)}
LEAST = {k: (bk, ks, 1) for k, (bk, ks, _) in TILES.items()}


def chain(tile, K, kb, splits):
    """MFMAs of 2 k in the longest chain of additions, from the loop structure: every split's slabs in order, a wave's
    share of each, its MFMAs dealt to the accumulators in turn."""
    bk, ks, accs = tile
    spans = [(r * K + k, min(bk, K - k)) for r in range(kb) for k in range(0, K, bk)]
    per, share = -(-len(spans) // splits), bk // ks
    longest = 0
    for s in range(0, len(spans), per):
        full = sum(share if n == bk or kb > 1 or splits > 1 else min(share, n) for _, n in spans[s:s + per])
        longest = max(longest, -(-full // (2 * accs)))
    return longest


def products(n, seed):
    rng = random.Random(seed)

    def lg(a, b):
        return round(math.exp(rng.uniform(math.log(a), math.log(b))))
    for _ in range(n):
        B, K, N = lg(1, 4096), lg(1, 9000), lg(1, 9000)
        yield rng, rng.choice([(N, B, K), (K, B, N), (N, K, B)])


def test_no_longer_chains_of_additions(planner):
    for rng, (M, N, K) in products(4000, 1):
        kb, batch = rng.choice([(1, 1), (1, 1), (1, 4), (35, 4)])
        cap = rng.choice([planner.ROOM, 0, 1 << 20])
        plan, (lkind, ls) = planner.f32(M, N, K, kb, batch, cap)
        was = chain(LEAST[lkind], K, kb, ls)
        reg = [planner.reg("f32", form, M, N, K, cap) for form in range(3)] if (kb, batch) == (1, 1) else []
        for kind, s in [plan] + reg:
            got = chain(TILES[kind], K, kb, s)
            assert got <= was, ((M, N, K, kb, batch, cap), kind, s, got, lkind, ls, was)


def test_splits_fit_the_room(planner):
    for rng, (M, N, K) in products(4000, 2):
        cap = round(math.exp(rng.uniform(0, math.log(1 << 26))))
        plans = [planner.f32(M, N, K, 1, 1, cap)[0]] + [planner.reg("f32", form, M, N, K, cap) for form in range(3)]
        assert all(s == 1 or s * M * N <= cap for _, s in plans), (M, N, K, cap, plans)

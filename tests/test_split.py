"""The shares of a whole replay's waves (dqx_split): they cover every tile once, in order, and the fullest wave holds no more than the least
that any bound per width allows (no GPU needed)."""
import ctypes as C
import itertools
import random

import pytest

from paper_2602_08923_amd import binding as B


def split(rows, n, f32, tree, sgs, blocks, waves):
    flat = (C.c_uint32 * (4 * len(rows)))(*itertools.chain(*rows))
    got = (C.c_uint32 * (2 * (blocks * waves + 1)))()
    f = B.lib().dqx_split
    f.restype = None
    f(flat, C.c_uint32(len(rows)), C.c_uint32(n), C.c_int(f32), C.c_int(tree), C.c_uint32(sgs), C.c_uint32(blocks), C.c_uint32(waves), got)
    return [(got[2 * i], got[2 * i + 1]) for i in range(blocks * waves + 1)]


def costs(f32, tree, n):
    return (12, 14, 15, 15) if f32 or n <= 4 else (12, 20, 22, 15 if n <= 12 else 12) if tree else (12, 24, 26, 15)


def least_fullest(tiles, cost, waves):
    s = max(c for t, c in zip(tiles, cost) if t)
    while True:
        most = [s // c for c in cost]
        if all(m or not t for t, m in zip(tiles, most)) and sum(t / m for t, m in zip(tiles, most) if t) <= waves:
            return s, most
        s += 1


@pytest.mark.parametrize("seed", range(40))
def test_shares_cover_every_tile_once_and_the_fullest_is_small(seed):
    rng = random.Random(seed)
    f32, tree, n, sgs = rng.randint(0, 1), rng.randint(0, 1), rng.choice([2, 4, 5, 8, 16, 100]), rng.choice([1, 2, 4, 4])
    blocks, waves = rng.choice([1, 3, 16, 100]), rng.choice([4, 8])
    paths = rng.choice([1, 2, 8, 61])
    size = max(1, int(blocks * waves * sgs * rng.choice([0.2, 1.0, 1.3, 2.5, 9.7]) / paths))
    rows = []
    for _ in range(paths):  # a chunk: mostly of one or two widths, sometimes empty of all
        a = rng.randint(0, size)
        row = [0, 0, 0, 0]
        for k in (a, size - a):
            row[rng.randint(0, 3)] += k if rng.random() < .9 else 0
        rows.append(row)
    if not any(map(sum, rows)):
        rows[0][1] = 5
    order = [(p, t, w) for p, row in enumerate(rows)
             for t, w in enumerate(itertools.chain.from_iterable([w] * -(-k // sgs) for w, k in enumerate(row)))]
    shares = split(rows, n, f32, tree, sgs, blocks, waves)
    place = {(p, t): i for i, (p, t, _) in enumerate(order)}
    place[(len(rows), 0)] = len(order)
    at = [place[s] for s in shares]          # every share begins at a tile, or at the end
    assert at[0] == 0 and at[-1] == len(order) and at == sorted(at)
    c = costs(f32, tree, n)
    tiles = [sum(1 for x in order if x[2] == w) for w in range(4)]
    least, most = least_fullest(tiles, c, blocks * waves)
    for lo, hi in zip(at, at[1:]):
        held = [sum(1 for x in order[lo:hi] if x[2] == w) for w in range(4)]
        if sum(1 for k in held if k) == 1:   # within the most of its width
            assert all(k <= m for k, m in zip(held, most)), (held, most)
        # at an edge between widths: one tile of either may be begun
        assert sum(k * x for k, x in zip(held, c)) <= least + 2 * max(c)


def chunks(by_width, n):
    """A bucket's chunks, super-groups by width of each."""
    m, edges = sum(by_width) // n, [0, *itertools.accumulate(by_width)]
    return [[max(0, min(hi, (c + 1) * m) - max(lo, c * m)) for lo, hi in zip(edges, edges[1:])] for c in range(n)]


def held_by_waves(rows, shares, sgs=4):
    """Tiles by width of every wave."""
    flat, first = [], []
    for row in rows:
        first.append(len(flat))
        flat += itertools.chain.from_iterable([w] * -(-k // sgs) for w, k in enumerate(row))
    at = [first[p] + t if p < len(rows) else len(flat) for p, t in shares]
    return [[flat[lo:hi].count(w) for w in range(4)] for lo, hi in zip(at, at[1:])]


@pytest.mark.parametrize("tree,n,blocks,waves,by_width,most", [(0, 24, 1280, 4, (5354, 9868, 5525, 10261), 3), (1, 2, 512, 8, (12249, 12534, 880, 8941), 2)])
def test_raw_tiles_are_dearer_than_two_bit_ones(tree, n, blocks, waves, by_width, most):
    """At equal cost the waves held one more: 18 and 8 % slower than with shares of equal counts."""
    rows = chunks(by_width, n)
    held = held_by_waves(rows, split(rows, n, 0, tree, 4, blocks, waves))
    assert max(h[3] for h in held) <= most and max(map(sum, held)) <= 3


def test_a_schedule_beyond_32_bits_of_cost():
    rows = [[2 ** 30, 2 ** 29, 2 ** 29 + 3, 7]]
    shares = split(rows, 8, 0, 0, 4, 256, 4)
    assert shares[0] == (0, 0) and shares[-1] == (1, 0)
    tiles = 2 ** 28 + 2 ** 27 + 2 ** 27 + 1 + 2
    starts = [t for _, t in shares[:-1]] + [tiles]
    assert starts == sorted(starts) and max(b - a for a, b in zip(starts, starts[1:])) < 2.2 * tiles / 1024

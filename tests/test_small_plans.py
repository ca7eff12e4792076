"""Launches too small to give every compute unit a long span: the number of spans is chosen by the cost of their pieces."""
import os
import random
import re

import pytest


@pytest.fixture(scope="module")
def b():
    from paper_2601_20499_amd import binding
    return binding


@pytest.mark.parametrize("seed", range(8))
def test_small_launches_are_cut_consistently(b, seed):
    """One head to 64, one query to several tiles, empty to 40-tile histories: pieces tile the spans and units (the kernel's
    own walk), no span is shorter than four tiles unless there is only one, and the same call gives the same plan."""
    rng = random.Random(seed)
    for _ in range(60):
        H, Nq, Nc = rng.choice([1, 2, 5, 12, 40, 64]), rng.choice([1, 64, 255, 256, 257, 600, 1170]), rng.choice([1, 64, 65, 300])
        lens = [rng.choice([0, 0, 1, 63, 64, 65, 500, 2560]) for _ in range(H)]
        sinks = [rng.choice([0, n, n // 3]) for n in lens]
        r = b.df_attn_plan(Nq, Nc, lens, sinks)
        assert r["consistent"] == 1 and 1 <= r["workgroups"] <= 256, (H, Nq, Nc, lens, r)
        assert r["span_max"] - r["span_min"] <= 1 and (r["n_teams"] == 1 or r["span_min"] >= 4), (H, Nq, Nc, lens, r)
        assert r["gives"] <= r["n_teams"] and r["line_len"] == r["n_groups"] * r["total_cols"]
        assert r == b.df_attn_plan(Nq, Nc, lens, sinks)


def test_short_units_are_not_cut(b):
    """Three heads of four tiles and one of one: three workgroups with whole units each, where spans of eight tiles had
    one workgroup walk all four units."""
    r = b.df_attn_plan(64, 64, [192, 192, 192, 0], [64, 64, 64, 0])
    assert r["workgroups"] == 3 and r["gives"] == 0 and r["pieces"] == 4


@pytest.mark.parametrize("Nq,Nc,lens,sinks,n_teams", [
    (1170, 4680, [9360] * 12, [1560] * 12, 48),   # 12 equal units, 51 spans fit: four spans a unit
    (237, 948, [4740] * 12, [316] * 12, 180),     # 256 fit: fifteen spans of six tiles a unit
    (4680, 4680, [9360] * 12, [1560] * 12, 13),   # spans of more than 64 tiles: all that the machine holds
])
def test_spans_that_fit_the_units(b, Nq, Nc, lens, sinks, n_teams):
    """Spans of less than 64 tiles are cut where the units end if a number near the largest does so."""
    r = b.df_attn_plan(Nq, Nc, lens, sinks)
    assert r["consistent"] == 1 and r["n_teams"] == n_teams, r


def constant(name):
    src = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_20499_amd", "csrc", "df_attn.hip")).read()
    return float(re.search(name + r" = ([\d.]+)f?\b", src)[1])


def cost(units, n):
    """Time of the slowest workgroup for n spans over units of so many tiles, span by span: pieces and what they cost besides
    their tiles; a unit's earlier pieces are there once the last of their workgroups has left its sums."""
    piece_cost, give, poll, fold, span_cost = (constant(f"k{x}Cost") for x in ("Piece", "Give", "Poll", "Fold", "Span"))
    line = sum(units)
    starts = [sum(units[:i]) for i in range(len(units) + 1)]
    cuts = [k * line // n for k in range(n + 1)]
    given = [[] for _ in units]                # when the pieces of a unit that are handed on are in memory
    worst = 0.0
    for lo, hi in zip(cuts, cuts[1:]):
        t, after = 0.0, None
        for u, (a, b) in enumerate(zip(starts, starts[1:])):
            if a < hi and b > lo:
                piece = piece_cost + min(hi, b) - max(lo, a)
                t += piece
                if b > hi:
                    t += give
                    given[u].append(piece + give)
                elif given[u]:
                    after = u
        worst = max(worst, t if after is None else max(t, max(given[after])) + poll + fold * len(given[after]))
    return (1 + span_cost * n) * worst


LAUNCHES = [    # queries, chunk, histories, sinks: the fewest spans of a length are much cheaper than their neighbours
    (754, 754, [377] + [3393] * 4 + [0], [377] * 5 + [0]),
    (362, 362, [3801] * 4 + [181] * 2 + [0] + [3801] * 3, [181] * 6 + [0] + [181] * 3),
    (321, 321, [107, 0, 0, 0] + [2247] * 8 + [107, 107, 2247, 107, 2247, 107, 107] + [2247] * 5, [107, 0, 0, 0] + [107] * 20),
]
rng = random.Random(31)
for _ in range(24):
    H, T, F = rng.choice([2, 5, 12, 24, 40]), rng.randint(60, 500), rng.choice([1, 3, 9, 21])
    frames = [rng.choice([0, 1, F, F]) for _ in range(H)]
    LAUNCHES.append((rng.choice([T, T // 4]), T * rng.choice([1, 3]), [f * T for f in frames], [T if f else 0 for f in frames]))


@pytest.mark.parametrize("Nq,Nc,lens,sinks", LAUNCHES)
def test_number_of_spans_is_the_cheapest_of_those_looked_at(b, Nq, Nc, lens, sinks):
    """No number that is always looked at costs less than the chosen one (by a share, for the fewest spans of a length)."""
    r = b.df_attn_plan(Nq, Nc, lens, sinks)
    tiles = lambda n: -(-n // 64)
    units = sorted((tiles(s) + tiles(l - s) + tiles(Nc) for l, s in zip(lens, sinks)), reverse=True) * r["n_groups"]
    line, most = r["line_len"], 256 // r["team_size"]
    assert line == sum(units)
    if line >= 64 * most:
        assert r["n_teams"] == most
        return
    n_max = max(1, min(most, line // 4))
    chosen = cost(units, r["n_teams"]) * (1 - 1e-5)        # the library counts in 32 bits
    for n in {n_max * e // 8 or 1 for e in range(4, 9)} | {n for n in range(n_max // len(units) * len(units), 0, -len(units))[:8]}:
        assert chosen <= cost(units, n), n
    for longer in (1, 2, 4, 6):
        n = max(1, line // (line // n_max + longer))
        assert chosen * constant("kSurelyCheaper") <= cost(units, n), n

"""Launches too small to give every compute unit a long span: the number of spans is chosen by the cost of their pieces."""
import random

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

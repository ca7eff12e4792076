"""What a call returns when a workgroup of its launch never gets to run: the waits for what it should have left behind
are bounded, and every result that needed it is NaN.  DF_ATTN_LOST_FLAG lets the reader of one flag give up at once."""
import numpy as np
import pytest
import torch

from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

TILE_K, N_CU = 64, 256


@pytest.fixture(scope="module")
def df():
    from paper_2601_20499_amd import binding
    return binding


class Call:
    """One launch of df_attn_fwd with every output, or one of df_head_score on the same inputs."""

    def __init__(self, df, H, d, Nq, Nc, lens, sinks):
        self.df, self.H, self.d, self.Nq, self.Nc, self.lens, self.sinks = df, H, d, Nq, Nc, lens, sinks
        dev = gu.dev()
        g = torch.Generator(device=dev).manual_seed(Nq + d)
        rnd = lambda *s: torch.randn(*s, generator=g, device=dev).to(torch.bfloat16)
        self.off = [0] + np.cumsum(lens).tolist()
        self.q, self.kc, self.vc = rnd(Nq, H, d), rnd(Nc, H, d), rnd(Nc, H, d)
        self.kh, self.vh = rnd(max(self.off[-1], 1), d), rnd(max(self.off[-1], 1), d)
        self.ws = torch.empty(df.df_attn_workspace_bytes(H, d, Nq), dtype=torch.uint8, device=dev)
        self.plan = df.df_attn_plan(Nq, Nc, lens, sinks)

    def attention(self):
        dev = gu.dev()
        out = torch.zeros(self.Nq, self.H, self.d, dtype=torch.bfloat16, device=dev)
        F, lse = torch.zeros(self.H, 3, device=dev), torch.zeros(self.H, self.Nq, device=dev)
        self.df.df_attn_fwd(self.q, self.kc, self.vc, self.kh, self.vh, self.off, self.sinks, out, self.d ** -0.5, lse_out=lse,
                            score_out=F, workspace=self.ws)
        torch.cuda.synchronize()
        return out, lse, F

    def scores(self):
        F = torch.zeros(self.H, 3, device=gu.dev())
        self.df.df_head_score(self.q, self.kc, self.kh, self.off, self.sinks, F, self.d ** -0.5, q_sample_stride=1, workspace=self.ws)
        torch.cuda.synchronize()
        return (F,)

    def cut_into(self, score):
        """Queries of a unit, workgroups of a team and number of teams of the launch, and of its units in three pieces or more (head, query
        tile of the last member, first span, last span)."""
        order = sorted(range(self.H), key=lambda h: -self.lens[h])
        rows, pieces = self.df.df_attn_units(self.d, score, self.Nq, self.Nc, self.lens, self.sinks)
        if rows:
            tiles, span, cut = -(-self.Nq // rows), 0, []
            for h in order:
                cut.append((h, tiles - 1, span, span + pieces[h] - 1))
                span += pieces[h]
            return rows, tiles, span, [c for c in cut if c[3] - c[2] >= 2]
        tiles = lambda n: -(-n // TILE_K)
        cols = [tiles(self.sinks[h]) + tiles(self.lens[h] - self.sinks[h]) + tiles(self.Nc) for h in order]
        line, n, team = self.plan["line_len"], self.plan["n_teams"], self.plan["team_size"]
        assert sum(cols) == self.plan["total_cols"]
        begin = [s * line // n for s in range(n + 1)]
        cut = []
        for grp in range(self.plan["n_groups"]):
            lo = grp * sum(cols)
            for h, c in zip(order, cols):
                spans = [s for s in range(n) if begin[s] < lo + c and begin[s + 1] > lo]
                cut.append((h, grp * team + team - 1, spans[0], spans[-1]))
                lo += c
        return 256, team, n, [c for c in cut if c[3] - c[2] >= 2]


# three heads, one of them without history, and two query tiles of 256, the second one ragged: a small launch whose teams are
# single workgroups in spans, and one whose teams are two
SMALL = dict(H=3, Nq=300, Nc=130, lens=[2500, 0, 1900], sinks=[100, 0, 64])
TEAMS = dict(H=3, Nq=300, Nc=130, lens=[25000, 0, 19000], sinks=[100, 0, 64])


@pytest.mark.parametrize("d,shape,team_size", [(64, SMALL, 1), (128, SMALL, 1), (128, TEAMS, 2)])
@pytest.mark.parametrize("which", ["first", "middle", "nearest"])
@pytest.mark.parametrize("score", [False, True])
def test_rows_of_a_unit_with_a_lost_piece_are_nan(df, monkeypatch, cut, d, shape, team_size, which, score):
    """One earlier piece of one unit, whichever is folded first, last or between: of the unit's rows, and through them the head's scores,
    nothing else is NaN."""
    call = Call(df, d=d, **shape)
    unit_rows, team, _, units = call.cut_into(score)
    assert df.df_attn_units(d, score, call.Nq, call.Nc, call.lens, call.sinks)[0] == cut
    if cut == 0:
        assert call.plan["team_size"] == team == team_size
    h, qt, first, last = max(units, key=lambda u: u[3] - u[2])
    span = {"first": first, "middle": (first + last) // 2, "nearest": last - 1}[which]
    rows = slice(qt * unit_rows, (qt + 1) * unit_rows)
    launch = call.scores if score else call.attention
    whole = launch()
    print(f"cut {cut} d {d} score {score} head {h} query tile {qt} spans {first} to {last}: lost {span}", flush=True)
    monkeypatch.setenv("DF_ATTN_LOST_FLAG", str(span * team + team - 1))
    lost = launch()
    others = [i for i in range(call.H) if i != h]
    assert torch.isnan(lost[-1][h]).all() and torch.equal(lost[-1][others], whole[-1][others])
    if not score:
        out, lse, _ = lost
        assert torch.isnan(lse[h, rows]).all() and torch.isnan(out[rows, h].float()).all()
        rest = torch.ones_like(lse, dtype=torch.bool)
        rest[h, rows] = False
        assert torch.equal(lse[rest], whole[1][rest]) and torch.equal(out[rest.t()], whole[0][rest.t()])
    monkeypatch.delenv("DF_ATTN_LOST_FLAG")        # what the launch left in the workspace does not touch the next one
    for a, b in zip(launch(), whole):
        assert torch.equal(a, b)


@pytest.mark.parametrize("score", [False, True])
def test_scores_are_nan_when_a_workgroup_never_says_it_is_done(df, monkeypatch, cut, score):
    call = Call(df, d=128, **SMALL)
    rows, team, teams, _ = call.cut_into(score)
    assert df.df_attn_units(128, score, call.Nq, call.Nc, call.lens, call.sinks)[0] == cut and teams * team > 2
    launch = call.scores if score else call.attention
    whole = launch()
    for wg in (0, teams * team - 1):
        monkeypatch.setenv("DF_ATTN_LOST_FLAG", str(N_CU + wg))
        lost = launch()
        assert torch.isnan(lost[-1]).all()
        assert all(torch.equal(a, b) for a, b in zip(lost[:-1], whole[:-1]))
        monkeypatch.delenv("DF_ATTN_LOST_FLAG")
        for a, b in zip(launch(), whole):
            assert torch.equal(a, b)


@pytest.mark.parametrize("d", [64, 128])
def test_a_single_team_waits_for_no_workgroup(df, monkeypatch, d):
    """Two or three workgroups that share no unit: whatever compute units they get, and one after the other if need be."""
    call = Call(df, d=d, H=1, Nq=300, Nc=40, lens=[100], sinks=[30])
    assert call.plan["n_teams"] == 1 and call.plan["workgroups"] == 2 and call.plan["cut_units"] == 0
    for way, units in (("spans", (0, [0])), ("128", (128, [1]))):
        monkeypatch.setenv("DF_ATTN_CUT", way)
        for score in (False, True):
            assert df.df_attn_units(d, score, 300, 40, [100], [30]) == units
        whole = call.attention() + call.scores()
        for flag in (0, 1, 2, N_CU, N_CU + 1, N_CU + 2):
            monkeypatch.setenv("DF_ATTN_LOST_FLAG", str(flag))
            for a, b in zip(call.attention() + call.scores(), whole):
                assert torch.isfinite(a.float()).all() and torch.equal(a, b)
        monkeypatch.delenv("DF_ATTN_LOST_FLAG")

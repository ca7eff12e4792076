"""What a call returns when a workgroup of its launch never gets to run: the waits for what it should have left behind
are bounded, and every result that needed it is NaN.  DF_ATTN_LOST_FLAG lets the reader of one flag give up at once."""
import numpy as np
import pytest
import torch

from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

TILE_Q, TILE_K, N_CU = 256, 64, 256


@pytest.fixture(scope="module")
def df():
    from paper_2601_20499_amd import binding
    return binding


class Call:
    """One launch of df_attn_fwd with every output and one of df_head_score on the same inputs."""

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

    def __call__(self):
        dev, scale = gu.dev(), self.d ** -0.5
        out = torch.zeros(self.Nq, self.H, self.d, dtype=torch.bfloat16, device=dev)
        F, F2 = torch.zeros(self.H, 3, device=dev), torch.zeros(self.H, 3, device=dev)
        lse = torch.zeros(self.H, self.Nq, device=dev)
        self.df.df_attn_fwd(self.q, self.kc, self.vc, self.kh, self.vh, self.off, self.sinks, out, scale, lse_out=lse,
                            score_out=F, workspace=self.ws)
        self.df.df_head_score(self.q, self.kc, self.kh, self.off, self.sinks, F2, scale, q_sample_stride=1, workspace=self.ws)
        torch.cuda.synchronize()
        return out, lse, F, F2

    def most_cut_unit(self):
        """(head, group of query tiles, first span, last span) of the unit that most spans share."""
        tiles = lambda n: -(-n // TILE_K)
        order = sorted(range(self.H), key=lambda h: -self.lens[h])
        cols = [tiles(self.sinks[h]) + tiles(self.lens[h] - self.sinks[h]) + tiles(self.Nc) for h in order]
        line, n = self.plan["line_len"], self.plan["n_teams"]
        assert sum(cols) == self.plan["total_cols"]
        begin = [s * line // n for s in range(n + 1)]
        best = None
        for grp in range(self.plan["n_groups"]):
            lo = grp * sum(cols)
            for h, c in zip(order, cols):
                spans = [s for s in range(n) if begin[s] < lo + c and begin[s + 1] > lo]
                if best is None or len(spans) > best[3] - best[2] + 1:
                    best = (h, grp, spans[0], spans[-1])
                lo += c
        return best


# three heads, one of them without history, and two query tiles, the second one ragged: a small launch whose teams are
# single workgroups, and one whose teams are two
SMALL = dict(H=3, Nq=300, Nc=130, lens=[2500, 0, 1900], sinks=[100, 0, 64])
TEAMS = dict(H=3, Nq=300, Nc=130, lens=[25000, 0, 19000], sinks=[100, 0, 64])


@pytest.mark.parametrize("d,shape,team_size", [(64, SMALL, 1), (128, SMALL, 1), (128, TEAMS, 2)])
@pytest.mark.parametrize("which", ["first", "middle", "nearest"])
def test_rows_of_a_unit_with_a_lost_piece_are_nan(df, monkeypatch, d, shape, team_size, which):
    call = Call(df, d=d, **shape)
    assert call.plan["team_size"] == team_size
    h, grp, first, last = call.most_cut_unit()
    assert last - first >= 2                       # three pieces or more: the flags lie in different lanes of the vote
    span = {"first": first, "middle": (first + last) // 2, "nearest": last - 1}[which]
    assert which != "middle" or first < span
    member = team_size - 1
    rows = slice((grp * team_size + member) * TILE_Q, (grp * team_size + member + 1) * TILE_Q)
    whole = call()
    monkeypatch.setenv("DF_ATTN_LOST_FLAG", str(span * team_size + member))
    out, lse, F, F2 = call()
    assert torch.isnan(lse[h, rows]).all() and torch.isnan(out[rows, h].float()).all()
    assert torch.isnan(F[h]).all() and torch.isnan(F2[h]).all()
    rest = torch.ones_like(lse, dtype=torch.bool)
    rest[h, rows] = False
    assert torch.equal(lse[rest], whole[1][rest]) and torch.equal(out[rest.t()], whole[0][rest.t()])
    others = [i for i in range(call.H) if i != h]
    assert torch.equal(F[others], whole[2][others]) and torch.equal(F2[others], whole[3][others])
    monkeypatch.delenv("DF_ATTN_LOST_FLAG")        # what the launch left in the workspace does not touch the next one
    for a, b in zip(call(), whole):
        assert torch.equal(a, b)


def test_scores_are_nan_when_a_workgroup_never_says_it_is_done(df, monkeypatch):
    call = Call(df, d=128, **SMALL)
    assert call.plan["workgroups"] > 2
    whole = call()
    monkeypatch.setenv("DF_ATTN_LOST_FLAG", str(N_CU + call.plan["workgroups"] - 1))
    out, lse, F, F2 = call()
    assert torch.isnan(F).all() and torch.isnan(F2).all()
    assert torch.equal(out, whole[0]) and torch.equal(lse, whole[1])
    monkeypatch.delenv("DF_ATTN_LOST_FLAG")
    for a, b in zip(call(), whole):
        assert torch.equal(a, b)


@pytest.mark.parametrize("d", [64, 128])
def test_a_single_team_waits_for_no_workgroup(df, monkeypatch, d):
    """Two workgroups that share no unit: whatever compute units they get, and one after the other if need be."""
    call = Call(df, d=d, H=1, Nq=300, Nc=40, lens=[100], sinks=[30])
    assert call.plan["n_teams"] == 1 and call.plan["workgroups"] == 2 and call.plan["cut_units"] == 0
    whole = call()
    for flag in (0, 1, N_CU, N_CU + 1):
        monkeypatch.setenv("DF_ATTN_LOST_FLAG", str(flag))
        for a, b in zip(call(), whole):
            assert torch.isfinite(a.float()).all() and torch.equal(a, b)

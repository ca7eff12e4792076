"""Keys that every query scores minus infinity have no weight, wherever they lie: a whole key tile of them may be the
first tile of a unit, or of a piece of a unit that several workgroups share, where the row has no reference yet."""
import pytest
import torch

from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

TILE = 64


@pytest.fixture(scope="module")
def df():
    from paper_2601_20499_amd import binding
    return binding


# tiles of the history (one head, 64 queries): a unit of 14 tiles cut twice in spans, one of 4 in one piece
@pytest.mark.parametrize("d,tiles,n_teams", [(128, 13, 3), (64, 13, 3), (128, 3, 1)])
@pytest.mark.parametrize("hand_over", ["1", "0"])
def test_a_tile_of_minus_infinity_scores(df, monkeypatch, cut, d, tiles, n_teams, hand_over):
    monkeypatch.setenv("DF_ATTN_HANDOVER", hand_over)
    dev, Nq, n = gu.dev(), 64, TILE * tiles
    rows, pieces = df.df_attn_units(d, False, Nq, TILE, [n], [TILE])
    assert rows == cut
    if cut:
        assert (pieces[0] > 1) == (tiles == 13), pieces
    else:
        assert df.df_attn_plan(Nq, TILE, [n], [TILE])["n_teams"] == n_teams
    g = torch.Generator(device=dev).manual_seed(d + tiles)
    rnd = lambda *s: torch.randn(*s, generator=g, device=dev).to(torch.bfloat16)
    q, kc, vc, k, vh = rnd(Nq, 1, d), rnd(TILE, 1, d), rnd(TILE, 1, d), rnd(n, d), rnd(n, d)
    q[:, :, 0] = 1
    ws = torch.empty(df.df_attn_workspace_bytes(1, d, Nq), dtype=torch.uint8, device=dev)
    # one tile, two that follow each other (the first two of the unit or of a piece among them), all but the chunk
    for first, last in [(t, t + 1) for t in range(tiles)] + [(t, t + 2) for t in range(tiles - 1)] + [(0, tiles)]:
        kh = k.clone()
        kh[TILE * first:TILE * last, 0] = float("-inf")
        out = torch.full_like(q, float("nan"))
        F, F2 = torch.full((1, 3), float("nan"), device=dev), torch.full((1, 3), float("nan"), device=dev)
        lse = torch.full((1, Nq), float("nan"), device=dev)
        df.df_attn_fwd(q, kc, vc, kh, vh, [0, n], [TILE], out, d ** -0.5, lse_out=lse, score_out=F, workspace=ws)
        df.df_head_score(q, kc, kh, [0, n], [TILE], F2, d ** -0.5, q_sample_stride=1, workspace=ws)
        torch.cuda.synchronize()
        logits = q[:, 0].double() @ torch.cat([kh, kc[:, 0]]).double().t() * d ** -0.5
        p = torch.softmax(logits, 1)
        what = f"tiles {first}..{last - 1}"
        gu.check_out(out[:, 0].double().cpu().numpy(), (p @ torch.cat([vh, vc[:, 0]]).double()).cpu().numpy(), what)
        assert (lse[0] - torch.logsumexp(logits, 1)).abs().max() <= gu.LSE_ABS, what
        R = torch.stack([p[:, :TILE].sum(), p[:, TILE:n].sum(), p[:, n:].sum()]) / Nq
        assert (F[0] - R).abs().max() <= gu.F_ABS and (F2[0] - R).abs().max() <= gu.F_ABS, what

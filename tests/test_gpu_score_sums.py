"""The two ways the per-head frame attention scores are summed - by the launch's first workgroup, or by the second
kernel when the workgroups of a launch cannot count on being on the device together - and the rows of units that are
finished in place, at the edges of query tiles and of the chunks the sums are read in."""
import numpy as np
import pytest
import torch

from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def df():
    from paper_2601_20499_amd import binding
    return binding


# (heads, d, queries, keys of the chunk): one query, one team; a ragged last tile; one tile more than a chunk of the
# sums holds at 64 heads (130 tiles at d = 128, 65 at d = 64, so two and three chunks); more units than workgroups, which are always
# cut into spans, the others as they are and in spans
@pytest.mark.parametrize("spans", [False, True])
@pytest.mark.parametrize("H,d,Nq,Nc", [(1, 128, 1, 1), (3, 64, 300, 65), (5, 128, 511, 200), (64, 128, 130 * 256 + 1, 33),
                                       (64, 64, 130 * 256 + 31, 33)])
def test_scores_and_rows_by_both_ways(df, monkeypatch, H, d, Nq, Nc, spans):
    if spans:
        monkeypatch.setenv("DF_ATTN_CUT", "spans")
    dev, n_sink, n_win = gu.dev(), 40, 70
    g = torch.Generator(device=dev).manual_seed(H * d + Nq)
    rnd = lambda *s: torch.randn(*s, generator=g, device=dev).to(torch.bfloat16)
    lens = [n_sink + n_win if h % 3 != 1 else 0 for h in range(H)]
    sink = [n_sink if n else 0 for n in lens]
    assert (df.df_attn_units(d, False, Nq, Nc, lens, sink)[0] == 0) == (spans or H == 64)
    off = [0] + np.cumsum(lens).tolist()
    q, kc, vc = rnd(Nq, H, d), rnd(Nc, H, d), rnd(Nc, H, d)
    kh, vh = rnd(off[-1], d), rnd(off[-1], d)
    ws = torch.empty(df.df_attn_workspace_bytes(H, d, Nq), dtype=torch.uint8, device=dev)

    def launch():
        out = torch.full((Nq + 1, H, d), float("nan"), dtype=torch.bfloat16, device=dev)     # one row that stays
        F, F2 = torch.full((H, 3), float("nan"), device=dev), torch.full((H, 3), float("nan"), device=dev)
        df.df_attn_fwd(q, kc, vc, kh, vh, off, sink, out[:Nq], d ** -0.5, score_out=F, workspace=ws)
        df.df_head_score(q, kc, kh, off, sink, F2, d ** -0.5, q_sample_stride=1, workspace=ws)
        torch.cuda.synchronize()
        assert torch.isnan(out[Nq].float()).all()
        return out[:Nq], F, F2

    first, again = launch(), launch()
    monkeypatch.setenv("DF_ATTN_HANDOVER", "0")
    second_kernel = launch()
    for a, b, c in zip(first, again, second_kernel):
        assert torch.equal(a, b) and torch.equal(a, c)
    out, F, F2 = first
    for h in range(0, H, max(1, H // 5)):
        keys = torch.cat([kh[off[h]:off[h + 1]], kc[:, h]]).double()
        p = torch.softmax(q[:, h].double() @ keys.t() * d ** -0.5, 1)
        ref = p @ torch.cat([vh[off[h]:off[h + 1]], vc[:, h]]).double()
        gu.check_out(out[:, h].double().cpu().numpy(), ref.cpu().numpy(), f"head {h}")
        s, n = sink[h], lens[h]
        R = torch.stack([p[:, :s].sum(), p[:, s:n].sum(), p[:, n:].sum()]) / Nq
        assert (F[h] - R).abs().max() <= gu.F_ABS and (F2[h] - R).abs().max() <= gu.F_ABS


@pytest.mark.parametrize("hand_over", ["1", "0"])
@pytest.mark.parametrize("d", [64, 128])
def test_sums_over_query_tiles_are_rounded_once(df, monkeypatch, d, hand_over):
    """The scores are those of the units' sums, which the launch leaves in the workspace ([H, query tiles, 4] floats), added up in 64 bits and
    rounded to 32 once: 131 of them in 32 bits are off by several times that."""
    monkeypatch.setenv("DF_ATTN_HANDOVER", hand_over)
    dev, H, tiles, Nc = gu.dev(), 5, 131, 33
    Nq, lens, sinks = 256 * (tiles - 1) + 7, [110, 0, 90, 300, 64], [40, 0, 90, 0, 1]
    off = [0] + np.cumsum(lens).tolist()
    g = torch.Generator(device=dev).manual_seed(d)
    rnd = lambda *s: torch.randn(*s, generator=g, device=dev).to(torch.bfloat16)
    q, kc, kh = rnd(Nq, H, d), rnd(Nc, H, d), rnd(off[-1], d)
    ws = torch.empty(df.df_attn_workspace_bytes(H, d, Nq), dtype=torch.uint8, device=dev)
    assert df.df_attn_units(d, True, Nq, Nc, lens, sinks)[0] == 0 and df.df_attn_units(d, False, Nq, Nc, lens, sinks)[0] == 0
    out, F, F2 = torch.empty_like(q), torch.empty(H, 3, device=dev), torch.empty(H, 3, device=dev)
    for score, launch in ((F, lambda: df.df_attn_fwd(q, kc, kc, kh, kh, off, sinks, out, d ** -0.5, score_out=F, workspace=ws)),
                          (F2, lambda: df.df_head_score(q, kc, kh, off, sinks, F2, d ** -0.5, q_sample_stride=1, workspace=ws))):
        launch()
        torch.cuda.synchronize()
        sums = ws[:H * tiles * 16].view(torch.float32).view(H, tiles, 4)[..., :2].double().sum(1)
        want = torch.stack([sums[:, 0], sums[:, 1] - sums[:, 0], Nq - sums[:, 1]], 1) / Nq
        # half a unit in the last place, and what 64 bits lose in differences
        assert ((score.double() - want).abs() <= 2.0 ** -24 * want.abs() + 1e-14).all(), ((score.double() - want) / want).abs().max()

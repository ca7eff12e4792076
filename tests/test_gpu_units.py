"""Launches that are cut unit by unit (workgroups of 256 queries, or of 128 whose two groups of waves halve every tile's keys): ragged and
single rows, tiles with keys for one half only, units in one piece and in many, every output, both ways to put pieces together; and the
same launches in spans."""
import numpy as np
import pytest
import torch

from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def df():
    from paper_2601_20499_amd import binding
    return binding


# queries, keys of the chunk, (sink, window) keys of the heads
CASES = [
    (1, 1, [(0, 0), (1, 0), (0, 1), (0, 65), (64, 64)]),   # one query, few keys
    (17, 31, [(1, 0), (0, 32), (33, 63), (0, 0)]),         # regions that end in a tile's first half, at it, behind it
    (64, 64, [(64, 128), (64, 128), (64, 128), (0, 0)]),   # half of the waves have rows
    (97, 65, [(0, 900), (64, 1700)]),                      # a wave with one row
    (128, 33, [(0, 5000)]),                                # one whole query tile, many pieces
    (129, 128, [(130, 1000), (0, 0), (0, 257)]),           # ... and one row more
    (300, 97, [(97, 1300), (0, 97), (97, 0), (0, 0), (0, 1300)]),
    (700, 350, [(0, 2000), (350, 0), (0, 0), (0, 350)] * 3),
    (1409, 96, [(65, 1500), (0, 33), (0, 0), (0, 33), (0, 0), (0, 33)] * 4),   # more units than fit with 128 queries each
]


@pytest.mark.parametrize("spans", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Nq,Nc,heads", CASES)
def test_every_output_by_both_ways(df, monkeypatch, d, Nq, Nc, heads, spans):
    if spans:
        monkeypatch.setenv("DF_ATTN_CUT", "spans")
    dev, H, scale = gu.dev(), len(heads), d ** -0.5
    sinks, lens = [s for s, _ in heads], [s + w for s, w in heads]
    units = df.df_attn_units(d, False, Nq, Nc, lens, sinks)
    print(f"d {d} Nq {Nq} Nc {Nc} heads {heads}: {units}, scores {df.df_attn_units(d, True, Nq, Nc, lens, sinks)}", flush=True)
    assert (units[0] == 0) == spans
    off = [0] + np.cumsum(lens).tolist()
    g = torch.Generator(device=dev).manual_seed(Nq + d)
    rnd = lambda *s: torch.randn(*s, generator=g, device=dev).to(torch.bfloat16)
    kc, vc = rnd(Nc, H, d), rnd(Nc, H, d)
    q = rnd(H, Nq, d).transpose(0, 1)                      # head-major rows
    kh, vh = rnd(max(off[-1], 1), d), rnd(max(off[-1], 1), d)
    ws = torch.full((df.df_attn_workspace_bytes(H, d, Nq),), 0xAB, dtype=torch.uint8, device=dev)

    def launch():
        out = torch.full((Nq + 1, H, d), float("nan"), dtype=torch.bfloat16, device=dev)     # one row that stays
        lse, F, F2 = torch.full((H, Nq), float("nan"), device=dev), torch.full((H, 3), float("nan"), device=dev), torch.zeros(H, 3, device=dev)
        df.df_attn_fwd(q, kc, vc, kh, vh, off, sinks, out[:Nq], scale, lse_out=lse, score_out=F, workspace=ws)
        df.df_head_score(q, kc, kh, off, sinks, F2, scale, q_sample_stride=1, workspace=ws)
        torch.cuda.synchronize()
        assert torch.isnan(out[Nq].float()).all()
        return out[:Nq], lse, F, F2

    first, again = launch(), launch()
    monkeypatch.setenv("DF_ATTN_HANDOVER", "0")
    for a, b, c in zip(first, again, launch()):
        assert torch.equal(a, b) and torch.equal(a, c)
    out, lse, F, F2 = first
    for h in range(H):
        logits = q[:, h].double() @ torch.cat([kh[off[h]:off[h + 1]], kc[:, h]]).double().t() * scale
        p = torch.softmax(logits, 1)
        ref = p @ torch.cat([vh[off[h]:off[h + 1]], vc[:, h]]).double()
        gu.check_out(out[:, h].double().cpu().numpy(), ref.cpu().numpy(), f"head {h}")
        assert (lse[h] - torch.logsumexp(logits, 1)).abs().max() <= gu.LSE_ABS
        s, n = sinks[h], lens[h]
        R = torch.stack([p[:, :s].sum(), p[:, s:n].sum(), p[:, n:].sum()]) / Nq
        assert (F[h] - R).abs().max() <= gu.F_ABS and (F2[h] - R).abs().max() <= gu.F_ABS


@pytest.mark.parametrize("Nq,lens,sinks", [(70, [70 + 210, 70, 0], [70, 70, 0]), (1300, [9000, 9000, 65], [63, 8937, 1])])
def test_without_scores_the_regions_are_one(df, Nq, lens, sinks):
    """Where the sink region ends does not matter then, down to the last bit."""
    dev, H, d = gu.dev(), 3, 128
    off = [0] + np.cumsum(lens).tolist()
    g = torch.Generator(device=dev).manual_seed(Nq)
    rnd = lambda *s: torch.randn(*s, generator=g, device=dev).to(torch.bfloat16)
    q, kc, vc, kh, vh = rnd(Nq, H, d), rnd(Nq, H, d), rnd(Nq, H, d), rnd(off[-1], d), rnd(off[-1], d)
    ws = torch.empty(df.df_attn_workspace_bytes(H, d, Nq), dtype=torch.uint8, device=dev)
    outs, lses = [torch.empty_like(q) for _ in range(2)], [torch.empty(H, Nq, device=dev) for _ in range(2)]
    for s, out, lse in zip((sinks, None), outs, lses):
        df.df_attn_fwd(q, kc, vc, kh, vh, off, s, out, d ** -0.5, lse_out=lse, workspace=ws)
    assert torch.equal(*outs) and torch.equal(*lses)
    for h in range(H):
        logits = q[:, h].double() @ torch.cat([kh[off[h]:off[h + 1]], kc[:, h]]).double().t() * d ** -0.5
        ref = torch.softmax(logits, 1) @ torch.cat([vh[off[h]:off[h + 1]], vc[:, h]]).double()
        gu.check_out(outs[0][:, h].double().cpu().numpy(), ref.cpu().numpy(), f"head {h}")
        assert (lses[0][h] - torch.logsumexp(logits, 1)).abs().max() <= gu.LSE_ABS


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Nq", [128, 300])
def test_replays_of_a_unit_in_many_pieces(df, cut, d, Nq):
    """By units every wave looks at every piece's flag and one puts them back, in spans one wave looks at all and puts them back: a
    replay, whose value is the same, waits again."""
    dev, lens, sinks = gu.dev(), [5000, 900], [0, 0]
    rows, pieces = df.df_attn_units(d, False, Nq, 33, lens, sinks)
    assert rows == cut
    assert (pieces[0] if cut else df.df_attn_plan(Nq, 33, lens, sinks)["max_pieces_per_unit"]) > 4
    g = torch.Generator(device=dev).manual_seed(d)
    rnd = lambda *s: torch.randn(*s, generator=g, device=dev).to(torch.bfloat16)
    q, kc, vc, kh, vh = rnd(Nq, 2, d), rnd(33, 2, d), rnd(33, 2, d), rnd(5900, d), rnd(5900, d)
    ws = torch.empty(df.df_attn_workspace_bytes(2, d, Nq), dtype=torch.uint8, device=dev)
    out, F = torch.empty_like(q), torch.empty(2, 3, device=dev)

    def step():
        df.df_attn_fwd(q, kc, vc, kh, vh, [0, 5000, 5900], sinks, out, d ** -0.5, score_out=F, workspace=ws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for replay in range(5):
        q.copy_(rnd(Nq, 2, d))
        vh.copy_(rnd(5900, d))
        step()
        torch.cuda.synchronize()
        want = out.clone(), F.clone()
        out.zero_()
        F.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[0]) and torch.equal(F, want[1]), replay

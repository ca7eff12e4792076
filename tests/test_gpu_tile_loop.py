"""The tile loop of the attention kernel where its special cases meet: regions of one to five tiles whose ends are less
than the load distance apart, ragged and whole last tiles, pieces of every length from one tile on, waves whose rows all
lie past the last query, and rows whose reference has to go up in the middle of a region."""
import numpy as np
import pytest
import torch

from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def df():
    from paper_2601_20499_amd import binding
    return binding


# queries; (sink, window) of the heads; keys of the chunk: one tile in all, one tile a region, no sink, no window, ends
# one to four tiles apart, whole and ragged last tiles (64 k - 1, 64 k, 64 k + 1)
SHAPES = [
    (1, [(0, 0)], 1),
    (33, [(1, 0), (0, 1)], 64),
    (300, [(64, 64), (0, 65), (63, 0)], 63),
    (257, [(1, 1), (65, 129), (128, 0), (0, 192)], 65),
    (511, [(127, 64), (192, 1), (64, 257), (0, 0), (320, 63)], 130),
    (97, [(256, 320), (64, 64)], 256),
]


@pytest.mark.parametrize("grows", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Nq,regions,Nc", SHAPES)
def test_regions_of_few_tiles(df, d, Nq, regions, Nc, grows):
    dev, H = gu.dev(), len(regions)
    g = torch.Generator(device=dev).manual_seed(100 * Nq + Nc + d)
    rnd = lambda *s: torch.randn(*s, generator=g, device=dev).to(torch.bfloat16)
    sink = [s for s, _ in regions]
    off = [0] + np.cumsum([s + w for s, w in regions]).tolist()
    q, kc, vc, kh, vh = rnd(Nq, H, d), rnd(Nc, H, d), rnd(Nc, H, d), rnd(off[-1], d), rnd(off[-1], d)
    if grows:
        # every eighth key outscores those before it: logits climb by about 2 sqrt(d) / 8 nats a key, through the
        # limit of the sums (2^100) several times in a region of a few hundred keys
        up = torch.full((d,), 1.0, device=dev).to(torch.bfloat16)
        q = (q.float() * 0.1 + up.float()).to(torch.bfloat16)
        for h in range(H):
            n = off[h + 1] - off[h]
            lift = lambda a, b: (0.25 * (torch.arange(a, b, device=dev) // 8)).to(torch.bfloat16)[:, None] * up
            kh[off[h]:off[h + 1]] += lift(0, n)
            kc[:, h] += lift(n, n + Nc)
    scale = d ** -0.5
    ws = torch.empty(df.df_attn_workspace_bytes(H, d, Nq), dtype=torch.uint8, device=dev)
    out = torch.full_like(q, float("nan"))
    F, F2 = torch.full((H, 3), float("nan"), device=dev), torch.full((H, 3), float("nan"), device=dev)
    lse = torch.full((H, Nq), float("nan"), device=dev)
    df.df_attn_fwd(q, kc, vc, kh, vh, off, sink, out, scale, lse_out=lse, score_out=F, workspace=ws)
    df.df_head_score(q, kc, kh, off, sink, F2, scale, q_sample_stride=1, workspace=ws)
    torch.cuda.synchronize()
    for h in range(H):
        logits = q[:, h].double() @ torch.cat([kh[off[h]:off[h + 1]], kc[:, h]]).double().t() * scale
        p = torch.softmax(logits, 1)
        ref = p @ torch.cat([vh[off[h]:off[h + 1]], vc[:, h]]).double()
        # one key may hold almost all of a row: the output is then a bf16 value times a bf16 P, up to two roundings of
        # 2^-9 of |V| <= 5
        err = (out[:, h].double() - ref).abs().max().item()
        assert np.isfinite(err) and err <= gu.MAX_ABS, (h, err)
        R = torch.logsumexp(logits, 1)
        # fp32 logits of up to |R|: products in fp32 (d roundings of 2^-24 in the worst case, a few in practice), c and the
        # reference rounded once each
        assert (lse[h] - R).abs().max() <= gu.LSE_ABS + 4e-6 * R.abs().max(), h
        s, n = sink[h], off[h + 1] - off[h]
        mass = torch.stack([p[:, :s].sum(), p[:, s:n].sum(), p[:, n:].sum()]) / Nq
        tol = gu.F_ABS + 4e-6 * logits.abs().max()                     # an error of a logit is one of its weight
        assert (F[h] - mass).abs().max() <= tol and (F2[h] - mass).abs().max() <= tol, h

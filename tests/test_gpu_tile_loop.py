"""The tile loop of the attention kernel where its special cases meet: regions of one to five tiles whose ends are less
than the load distance apart, ragged and whole last tiles, pieces of every length from one tile on, waves whose rows all
lie past the last query, and rows whose reference has to go up after a piece's first tile - by far, so that nothing of what
was summed before is left, and by so little that it keeps its share."""
import itertools
import math

import numpy as np
import pytest
import torch

from tests import gpu_util as gu
from tests import test_units


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
# how the logits go on from a row's first keys: by noise of about a nat alone; up by 2 sqrt(d) nats every eight keys, 185 (d =
# 64) or 261 bits a tile, past the limit of the sums (2^100) in every tile; up once, behind the unit's first tile, by 94 to 98 bits by
# wave, after which the sums pass the limit with one tile or a few that all have a share in them
GROWTH = ["none", "steep", "plateau"]


def inputs(d, Nq, regions, Nc, growth):
    """q, k_cur, v_cur, k_hist, v_hist (bf16, on the CPU) and the history offsets."""
    H = len(regions)
    g = torch.Generator().manual_seed(100 * Nq + Nc + d)
    rnd = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16)
    off = [0] + np.cumsum([s + w for s, w in regions]).tolist()
    q, kc, vc, kh, vh = rnd(Nq, H, d), rnd(Nc, H, d), rnd(Nc, H, d), rnd(off[-1], d), rnd(off[-1], d)
    if growth != "none":
        # q . (1, ..., 1) is about d: a lift of x is x sqrt(d) nats
        if growth == "steep":
            q = (q.float() * 0.1 + 1.0).to(torch.bfloat16)
        else:
            wave = (torch.arange(Nq) // 32)[:, None, None] + 3 * torch.arange(H)[:, None]
            q = ((q.float() * 0.02 + 1.0) * (94.5 + 0.5 * (wave % 8)) / 97).to(torch.bfloat16)
            kh, kc = kh * 0.25, kc * 0.25
        for h in range(H):
            n = off[h + 1] - off[h]
            i = torch.arange(n + Nc)
            first = next(min(x, 64) for x in (*regions[h], Nc) if x)
            lift = 2.0 * (i // 8) if growth == "steep" else (i >= first) * (97 * math.log(2) / d ** 0.5)
            lift = lift.to(torch.float32)[:, None]
            kh[off[h]:off[h + 1]] = (kh[off[h]:off[h + 1]].float() + lift[:n]).to(torch.bfloat16)
            kc[:, h] = (kc[:, h].float() + lift[n:]).to(torch.bfloat16)
    return q, kc, vc, kh, vh, off


def pieces_of(df, d, tiles, regions, Nq, Nc, cut):
    """Pieces of the launch: (head, queries, first tile, tile behind the last)."""
    lens, sinks = [s + w for s, w in regions], [s for s, _ in regions]
    rows, count = df.df_attn_units(d, False, Nq, Nc, lens, sinks)
    assert rows == cut
    if cut:
        ahead, lag = test_units.SHAPE[d, False, cut]
        for h, k in enumerate(count):
            n = len(tiles[h])
            length = -(-(n - ahead - test_units.begin(k - 1, k, 0, lag)) // k)
            starts = [test_units.begin(j, k, length, lag) for j in range(k)] + [n]
            yield from ((h, range(Nq), begin, end) for begin, end in zip(starts, starts[1:]))
        return
    plan = df.df_attn_plan(Nq, Nc, lens, sinks)
    order = sorted(range(len(regions)), key=lambda h: -sum(regions[h]))
    cuts = {k * plan["line_len"] // plan["n_teams"] for k in range(1, plan["n_teams"])}
    group_rows, at = plan["team_size"] * 256, 0
    for group, h in itertools.product(range(plan["n_groups"]), order):
        starts = [0] + [c - at for c in sorted(cuts) if at < c < at + len(tiles[h])]
        queries = range(group * group_rows, min(Nq, (group + 1) * group_rows))
        yield from ((h, queries, begin, end) for begin, end in zip(starts, starts[1:] + [len(tiles[h])]))
        at += len(tiles[h])


def raises(df, logits, regions, Nq, Nc, d, cut):
    """The rule for references on the pieces of the launch, from the logits of the heads in 64 bits: (raises after the first tile in which
    a wave has a key, of which some row's earlier tiles keep a hundredth of its sum, pieces of more than one tile)."""
    tiles = [[(r0 + a, r0 + min(a + 64, n)) for r0, n in ((0, s), (s, w), (s + w, Nc)) for a in range(0, n, 64)] for s, w in regions]
    n_raised = n_shared = n_long = 0
    for h, queries, begin, end in pieces_of(df, d, tiles, regions, Nq, Nc, cut):
        n_long += end - begin > 1
        for row0, first in itertools.product(queries[::32], (0, 32) if cut == 128 else (0,)):
            x = logits[h][row0:row0 + 32] * math.log2(math.e)
            ref, l = None, None
            for a, b in tiles[h][begin:end]:
                # where the two groups of waves halve the keys, a wave has 32 of a tile
                a, b = a + first, min(b, a + first + 32) if cut == 128 else b
                if a >= b:
                    continue
                if ref is None:
                    ref, l = x[:, a:b].amax(1), torch.zeros(len(x), 4, dtype=torch.float64)
                key = torch.arange(b - a) % 16              # quarter of the wave that holds a key of its block of 16
                quarter = (key // 8 * 2 + (key // 2 % 2 == 0) * 1)
                share = lambda r: torch.exp2(x[:, a:b] - r[:, None]) @ torch.nn.functional.one_hot(quarter, 4).double()
                new = l + share(ref)
                lanes = torch.zeros(32, 4, dtype=torch.float64)     # of the wave's two rows that a lane has
                lanes[:len(x)] = new
                if (lanes[:16] + lanes[16:]).max() > 2.0 ** 100:
                    up = torch.maximum(torch.maximum(x[:, a:b].amax(1), ref), ref + torch.log2(l.sum(1)))
                    l = l * torch.exp2(ref - up)[:, None]
                    before, ref, new = l.sum(1), up, l + share(up)
                    n_raised += 1
                    n_shared += bool((before > 0.01 * new.sum(1)).any())
                l = new
    return n_raised, n_shared, n_long


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Nq,regions,Nc", SHAPES)
def test_inputs_raise_references(df, cut, d, Nq, regions, Nc):
    """What the inputs of the GPU test below are made for, however the launch is cut: wherever a piece has a second tile, some reference
    goes up behind the first; and where units have three or more tiles, some time with earlier tiles that count."""
    for growth in GROWTH:
        q, kc, _, kh, _, off = inputs(d, Nq, regions, Nc, growth)
        logits = [q[:, h].double() @ torch.cat([kh[off[h]:off[h + 1]], kc[:, h]]).double().t() * d ** -0.5 for h in range(len(regions))]
        n_raised, n_shared, n_long = raises(df, logits, regions, Nq, Nc, d, cut)
        print(growth, n_raised, n_shared, n_long)
        if growth == "none":
            assert n_raised == 0
        elif growth == "steep":
            # 33 keys go up by 92 bits at d = 64: a wave with half of the keys of a tile and one before it stays below the limit
            assert (n_raised > 0) == (n_long > 0 and (cut, d, Nq) != (128, 64, 33))
        elif Nq > 33:
            assert n_shared > 1


@pytest.mark.gpu
@pytest.mark.parametrize("growth", GROWTH)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Nq,regions,Nc", SHAPES)
def test_regions_of_few_tiles(df, cut, d, Nq, regions, Nc, growth):
    dev, sink = gu.dev(), [s for s, _ in regions]
    *tensors, off = inputs(d, Nq, regions, Nc, growth)
    q, kc, vc, kh, vh = (t.to(dev) for t in tensors)
    assert df.df_attn_units(d, False, Nq, Nc, [s + w for s, w in regions], sink)[0] == cut
    check_against_reference(df, q, kc, vc, kh, vh, off, sink)


@pytest.mark.gpu
@pytest.mark.parametrize("stride", [16384, 40000])
@pytest.mark.parametrize("d", [64, 128])
def test_pieces_of_one_to_three_tiles_of_a_chunk_with_wide_rows(df, cut, d, stride):
    """Rows of the current chunk 32 KB and more apart, in pieces so short that the loop's first loads are of tiles that they do not
    have: offsets and descriptors of such tiles are not those of the chunk."""
    dev, regions, Nc = gu.dev(), [(0, 0), (65, 1), (1, 64), (0, 63)], 65
    q, kc, vc, kh, vh, off = inputs(d, 40, regions, Nc, "none")
    wide = torch.zeros(2, Nc, stride, dtype=torch.bfloat16, device=dev)
    rows = [x[:, :len(regions) * d].view(Nc, len(regions), d) for x in wide]
    rows[0].copy_(kc)
    rows[1].copy_(vc)
    assert rows[0].stride(0) == stride
    assert df.df_attn_units(d, False, 40, Nc, [s + w for s, w in regions], [s for s, _ in regions])[0] == cut
    check_against_reference(df, q.to(dev), *rows, kh.to(dev), vh.to(dev), off, [s for s, _ in regions])


def check_against_reference(df, q, kc, vc, kh, vh, off, sink):
    """Outputs, log-sum-exp and both kinds of scores against 64 bits."""
    (Nq, H, d), dev = q.shape, q.device
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
        # products summed in fp32 (d roundings of 2^-24 in the worst case, half of that allowed); an error of a logit is one of
        # its key's weight
        logit_err = 4e-6 * logits.abs().max().item()
        # one key may hold almost all of a row: the output is then a bf16 value times a bf16 P, up to two roundings of
        # 2^-9 of |V| <= 5
        err = (out[:, h].double() - ref).abs().max().item()
        assert np.isfinite(err) and err <= gu.MAX_ABS + 5 * logit_err, (h, err)
        R = torch.logsumexp(logits, 1)
        # fp32 logits of up to |R|, c and the reference rounded once each
        assert (lse[h] - R).abs().max() <= gu.LSE_ABS + 4e-6 * R.abs().max(), h
        s, n = sink[h], off[h + 1] - off[h]
        mass = torch.stack([p[:, :s].sum(), p[:, s:n].sum(), p[:, n:].sum()]) / Nq
        tol = gu.F_ABS + logit_err
        assert (F[h] - mass).abs().max() <= tol and (F2[h] - mass).abs().max() <= tol, h

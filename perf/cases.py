"""The work a generation loop has this library do, as cases that can be timed and compared.

A case is one call, or one short sequence of calls, through the public entry points of
paper_2601_20499_amd.binding.  Its fields:

    kind    attn     df_attn_fwd on a packed context
            step     df_attn_fwd on the rolling cache in place, then df_kv_append: one chunk-layer of a loop
            score    df_head_score on the un-pruned context of every head
            typing   df_head_score, the scores copied to the host, df_classify: how a layer's heads get their types
            pack     df_pack_context out of a rolling cache whose ring has wrapped
            append   df_kv_append to a full rolling cache
    d, T, chunk      head dimension, tokens per latent frame, frames per chunk (Nq = Nc = chunk * T)
    heads   "9x1/5 3x0/0" = nine heads with one sink frame and five window frames, three with no history
            (the contexts of the five head types: full s/w, sink s/0, neighbour 0/w, dummy 0/0, packed dummy 0/1)
    score, lse       whether df_attn_fwd also returns the fused frame attention scores / the log-sum-exp
    stride  df_head_score scores every stride-th query

The heads of the different groups are interleaved: a layer's dummy heads lie anywhere among the others.
"""
import torch

from paper_2601_20499_amd import binding as df

_DEVICE = "cuda"


def listed():
    def case(name, kind, T, heads, d=128, chunk=3, score=False, lse=False, stride=1):
        return dict(name=name, kind=kind, d=d, T=T, chunk=chunk, heads=heads, score=score, lse=lse, stride=stride)

    return [
        # the smallest call: a one-frame chunk of 64 tokens, four narrow heads, three cached frames; all latency
        case("attn_tiny_d64", "attn", 64, "3x1/2 1x0/0", d=64, chunk=1, score=True),
        # a quarter-resolution preview (390 tokens per frame): 1170 queries, all five head types, every output
        case("attn_preview", "attn", 390, "3x1/5 2x1/0 3x0/5 2x0/0 2x0/1", score=True, lse=True),
        # 832x480 chunk, a quarter of the heads dummy, context packed at the last re-typing, fused scores on
        case("attn_480p", "attn", 1560, "9x1/5 3x0/0", score=True),
        # the same geometry as the loop runs it once heads have their three types: the rolling cache read in
        # place, half of the heads packed dummies, then the chunk appended
        case("step_480p_dhp", "step", 1560, "2x1/0 4x0/5 6x0/1"),
        # a layer with 40 heads (14B-class geometry), same loop, heads of all types
        case("step_480p_40_heads", "step", 1560, "7x1/0 13x0/5 20x0/1"),
        # 1280x720 chunk with twelve cached frames
        case("attn_720p", "attn", 3600, "9x1/11 3x0/0", score=True),
        # 1920x1088 chunk: the largest launch, 24480 queries; inference without scores
        case("attn_1080p", "attn", 8160, "6x1/5 6x0/1"),
        # long video: histories of 3 to 60 frames side by side with dummy heads
        case("attn_long_context", "attn", 1560, "1x1/2 1x1/9 1x1/23 1x1/46 1x1/7 1x1/59 6x0/0"),
        # head programming of one layer at the start of a shot: a quarter of the queries, every head un-pruned
        case("score_480p", "score", 1560, "12x1/5", stride=4),
        # the same with 21 cached frames and the decision taken layer by layer on the host
        case("typing_480p_21_frames", "typing", 1560, "12x1/20", stride=4),
        # after heads were re-typed: their contexts gathered out of the rolling cache
        case("pack_480p", "pack", 1560, "9x1/5 3x0/0"),
        # a finished 1280x720 chunk goes into a full cache
        case("append_720p", "append", 3600, "9x1/11 3x0/0"),
    ]


def _contexts(case):
    """[(sink frames, window frames)] per head, groups interleaved."""
    groups = []
    for part in case["heads"].split():
        n, ctx = part.split("x")
        s, w = ctx.split("/")
        groups.append((int(n), int(s), int(w)))
    spread = [((i + 0.5) / n, g, s, w) for g, (n, s, w) in enumerate(groups) for i in range(n)]
    return [(s, w) for _, _, s, w in sorted(spread)]


def _sizes(case):
    """Queries (= keys of the chunk), per-head sink and window tokens."""
    ctx, T = _contexts(case), case["T"]
    return case["chunk"] * T, [s * T for s, _ in ctx], [w * T for _, w in ctx]


def draw(rng):
    most = work(next(c for c in listed() if c["name"] == "attn_1080p"))["flops"]
    while True:
        kind = rng.choice(["attn", "attn", "step", "score", "typing", "pack", "append"])
        d = rng.choice([64, 128, 128])
        T = int(round(2 ** rng.uniform(6, 13)))                # 64 ... 8192 tokens per frame, mostly odd sizes
        chunk = rng.choice([1, 2, 3, 3])
        H = rng.choice([2, 4, 5, 8, 12, 12, 16, 24, 40])
        frames = int(round(2 ** rng.uniform(1, 6)))            # cached frames of a full head: 2 ... 64
        if kind in ("score", "typing"):
            heads = "%dx1/%d" % (H, frames - 1)
        else:
            kinds = ["1/%d" % (frames - 1), "1/0", "0/%d" % (frames - 1), "0/0", "0/1"]
            picked = [rng.choice(kinds) for _ in range(H)]
            picked[rng.randrange(H)] = kinds[0]
            heads = " ".join("%dx%s" % (picked.count(k), k) for k in kinds if k in picked)
        case = dict(kind=kind, d=d, T=T, chunk=chunk, heads=heads, score=kind == "attn" and rng.random() < 0.5,
                    lse=kind == "attn" and rng.random() < 0.25, stride=4 if kind in ("score", "typing") else 1)
        w = work(case)
        if w["flops"] <= most and w["bytes"] <= 2e9 and chunk * T <= 32768:
            return case


def prepare(case, seed):
    Nq, sink, win = _sizes(case)
    H, d, kind, scale = len(sink), case["d"], case["kind"], case["d"] ** -0.5
    g = torch.Generator(device=_DEVICE).manual_seed(seed)

    def gauss(*shape):
        return torch.randn(*shape, generator=g, device=_DEVICE, dtype=torch.bfloat16)

    st = dict(kind=kind, scale=scale, stride=case["stride"])
    # Queries have a per-head mean; where a head leans on the current chunk (the heads with no or little history,
    # and a quarter of the heads while they are being scored) that chunk's keys are shifted along it.
    mean = 0.4 * torch.randn(H, d, generator=g, device=_DEVICE)
    q = (torch.randn(Nq, H, d, generator=g, device=_DEVICE) + mean).to(torch.bfloat16)
    n_dummy = max(1, H // 4)
    if kind in ("score", "typing"):
        lean = torch.zeros(H, device=_DEVICE)
        lean[torch.randperm(H, generator=g, device=_DEVICE)[:n_dummy]] = 2.0
    else:
        lean = torch.tensor([2.0 if sink[h] + win[h] <= case["T"] else 0.0 for h in range(H)], device=_DEVICE)
    k_cur = (torch.randn(Nq, H, d, generator=g, device=_DEVICE) + lean[:, None] * mean).to(torch.bfloat16)
    v_cur = gauss(Nq, H, d)
    st.update(q=q, k_cur=k_cur, v_cur=v_cur)
    rows = [s + w for s, w in zip(sink, win)]
    off = [0]
    for r in rows:
        off.append(off[-1] + r)
    n_rows = max(off[-1], 1)

    if kind in ("step", "pack", "append"):
        cache = df.Cache(gauss(n_rows, d), gauss(n_rows, d), off, sink, win, d)
        for h in range(H):                                  # a cache in the middle of a long video: full, ring wrapped
            cache.sink_len[h], cache.win_len[h] = sink[h], win[h]
            cache.win_pos[h] = (case["chunk"] * case["T"]) % win[h] if win[h] else 0
        st["cache"] = cache
    if kind in ("attn", "score", "typing"):
        st.update(k_hist=gauss(n_rows, d), off=off, sink=sink)
        if kind == "attn":
            st["v_hist"] = gauss(n_rows, d)
    if kind in ("attn", "step"):
        st["out"] = torch.empty_like(q)
        st["F"] = torch.empty(H, 3, device=_DEVICE) if case["score"] else None
        st["lse"] = torch.empty(H, Nq, device=_DEVICE) if case["lse"] else None
    if kind in ("score", "typing"):
        st["F"] = torch.empty(H, 3, device=_DEVICE)
        st["n_dummy"] = n_dummy
    if kind in ("attn", "step", "score", "typing"):
        st["ws"] = torch.empty(df.df_attn_workspace_bytes(H, d, Nq), dtype=torch.uint8, device=_DEVICE)
    if kind == "pack":
        st.update(take_sink=sink, take_win=win, k_pack=torch.zeros(n_rows, d, dtype=torch.bfloat16, device=_DEVICE),
                  v_pack=torch.zeros(n_rows, d, dtype=torch.bfloat16, device=_DEVICE))
    return st


def run(st):
    kind = st["kind"]
    if kind == "attn":
        df.df_attn_fwd(st["q"], st["k_cur"], st["v_cur"], st["k_hist"], st["v_hist"], st["off"], st["sink"], st["out"],
                       st["scale"], lse_out=st["lse"], score_out=st["F"], workspace=st["ws"])
        return [x for x in (st["out"], st["F"], st["lse"]) if x is not None]
    if kind == "step":
        cache = st["cache"]
        k, v, off, sink, length = cache.in_place()
        df.df_attn_fwd(st["q"], st["k_cur"], st["v_cur"], k, v, off, sink, st["out"], st["scale"], workspace=st["ws"],
                       hist_len=length)
        df.df_kv_append(cache, st["k_cur"], st["v_cur"])
        return [st["out"], k, v]
    if kind in ("score", "typing"):
        df.df_head_score(st["q"], st["k_cur"], st["k_hist"], st["off"], st["sink"], st["F"], st["scale"],
                         q_sample_stride=st["stride"], workspace=st["ws"])
        if kind == "score":
            return st["F"]
        types, keys = df.df_classify(st["F"].tolist(), st["n_dummy"], df.DF_CLASSIFY_TWO_CLASS)
        return [st["F"], torch.tensor(types), torch.tensor(keys)]
    if kind == "pack":
        off, sink = df.df_pack_context(st["cache"], st["take_sink"], st["take_win"], st["k_pack"], st["v_pack"])
        return [st["k_pack"], st["v_pack"], off[-1]]
    df.df_kv_append(st["cache"], st["k_cur"], st["v_cur"])
    return [st["cache"].k_cache, st["cache"].v_cache]


def _exact_attention(st, case):
    """Outputs, frame attention scores [H, 3] and log-sum-exp [H, Nq] of the queries in `st`, in 64 bits."""
    Nq, sink, win = _sizes(case)
    H, d, scale = len(sink), case["d"], st["scale"]
    if "cache" in st:
        k_hist, v_hist, off = st["cache"].k_cache, st["cache"].v_cache, list(st["cache"].head_row_off)
    else:
        k_hist, v_hist, off = st["k_hist"], st.get("v_hist"), st["off"]
    q, values = st["q"][:: case["stride"]], v_hist is not None
    n = q.shape[0]
    out = torch.empty(n, H, d, dtype=torch.float64, device=_DEVICE)
    F = torch.zeros(H, 3, dtype=torch.float64, device=_DEVICE)
    lse = torch.empty(H, n, dtype=torch.float64, device=_DEVICE)
    for h in range(H):
        keys = torch.cat([k_hist[off[h]:off[h] + sink[h] + win[h]], st["k_cur"][:, h]]).double()
        vals = torch.cat([v_hist[off[h]:off[h] + sink[h] + win[h]], st["v_cur"][:, h]]).double() if values else None
        rows = max(1, 100_000_000 // keys.shape[0])
        for r in range(0, n, rows):
            logits = (q[r:r + rows, h].double() @ keys.t()).mul_(scale)
            lse[h, r:r + rows] = torch.logsumexp(logits, 1)
            p = logits.sub_(lse[h, r:r + rows, None]).exp_()
            for i, part in enumerate((p[:, :sink[h]], p[:, sink[h]:sink[h] + win[h]], p[:, sink[h] + win[h]:])):
                F[h, i] += part.sum()
            if values:
                out[r:r + rows, h] = p @ vals
    return out, F / n, lse


def exact(case, seed):
    """What run returns, by plain torch in 64 bits; the copies (pack, append, the cache of a step) have no sums to compare."""
    kind = case["kind"]
    if kind in ("pack", "append"):
        return None
    st = prepare(case, seed)
    out, F, lse = _exact_attention(st, case)
    if kind == "attn":
        return [out] + [F] * case["score"] + [lse] * case["lse"]
    if kind == "step":
        return [out, None, None]
    if kind == "score":
        return F
    return [F, None, F[:, 0] + F[:, 1]]


def work(case):
    Nq, sink, win = _sizes(case)
    H, d, kind = len(sink), case["d"], case["kind"]
    rows = sum(sink) + sum(win)
    row = 2 * d                                              # bytes of one bf16 row
    moved, flops = 0.0, 0.0
    if kind in ("attn", "step"):
        moved += row * (2 * Nq * H + 2 * (rows + Nq * H))    # queries and outputs, keys and values
        moved += 12 * H * case["score"] + 4 * H * Nq * case["lse"]
        flops += 4.0 * Nq * d * (rows + Nq * H)
    if kind in ("score", "typing"):
        n = -(-Nq // case["stride"])
        moved += row * (n * H + rows + Nq * H) + 12 * H
        flops += 2.0 * n * d * (rows + Nq * H)
    if kind == "pack":
        moved += 4 * row * rows                              # keys and values, read and written
    if kind in ("step", "append"):
        moved += 4 * row * sum(min(Nq, w) for w in win)      # full sinks take nothing, a short window the last tokens
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    # Against the same path in 64 bits (every row of the small and of the 832x480 launches): outputs, which round the
    # probabilities and themselves to bf16, differ by up to rel 2.35e-3 and max 1.43e-2; scores and log-sum-exp, sums
    # in 32 bits over thousands of keys and queries, by up to rel 9e-8 and max 2e-7 (a longer serial order: ten times
    # that).
    if case["kind"] in ("pack", "append"):
        return "exact"
    if case["kind"] in ("score", "typing"):
        return {"rel": 2e-6, "max": 1e-5, "differ": 0.0}
    return {"rel": 1e-2, "max": 6e-2}

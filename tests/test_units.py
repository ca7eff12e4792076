"""Which launches are cut unit by unit, and into what (the host's choice; no GPU)."""
import ctypes
import os
import random
import re
import time

import pytest


@pytest.fixture(scope="module")
def b():
    from paper_2601_20499_amd import binding
    return binding


# By head dimension, scores only, queries of a unit: tiles that the last piece may have more than the one before it, and sixteenths of a
# tile that each of the others has more than the next.
SHAPE = {(128, False, 128): (3, 18), (128, False, 256): (1, 19), (64, False, 128): (4, 16), (64, False, 256): (2, 14),
         (128, True, 128): (3, 0), (128, True, 256): (1, 0), (64, True, 128): (4, 0), (64, True, 256): (2, 0)}


def begin(j, count, length, lag):
    return j * length + (j * (2 * count - 3 - j) // 2 * lag >> 4)


def tiles(n):
    return -(-n // 64)


def test_pieces_fit_the_machine_and_the_units(b):
    """Random mixes: all heads are cut or none, no piece is empty, all pieces have a compute unit, and no head has more pieces than one that
    is as long as the head with the longest needs."""
    rng, cut = random.Random(128), {128: 0, 256: 0}
    for _ in range(1500):
        H, d, score = rng.choice([1, 2, 5, 12, 40, 64]), rng.choice([64, 128]), rng.random() < 0.3
        Nq, Nc = rng.choice([1, 64, 65, 128, 129, 600, 1170, 4680]), rng.choice([1, 64, 300, 4680])
        lens = [rng.choice([0, 0, 1, 64, 65, 500, 2560, 30000]) for _ in range(H)]
        sinks = [rng.choice([0, n, n // 3]) for n in lens]
        rows, pieces = b.df_attn_units(d, score, Nq, Nc, lens, sinks)
        assert (rows, pieces) == b.df_attn_units(d, score, Nq, Nc, lens, sinks)
        if not rows:
            assert not any(pieces)
            continue
        cut[rows] += 1
        units = [tiles(s) + tiles(n - s) + tiles(Nc) for n, s in zip(lens, sinks)]
        assert all(1 <= k <= n for k, n in zip(pieces, units))
        assert sum(pieces) * -(-Nq // rows) <= 256
        ahead, lag = SHAPE[d, score, rows]
        lengths = []
        for n, k in zip(units, pieces):
            lengths.append(max(1, n - ahead) if k == 1 else -(-(n - ahead - begin(k - 1, k, 0, lag)) // k))
            starts = [begin(j, k, lengths[-1], lag) for j in range(k)] + [n]
            assert all(a < b for a, b in zip(starts, starts[1:]))
        longest = max(lengths)
        assert all(k == 1 or begin(k - 2, k - 1, longest, lag) + longest + ahead < n for n, k in zip(units, pieces))
    assert min(cut.values()) > 50


def launch_costs():
    """The constants of the model by head dimension, scores only, queries of a unit, from the source."""
    src = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_20499_amd", "csrc", "df_attn.hip")).read()
    body = src[src.index("constexpr LaunchCost kLaunchCost"):]
    sets = re.findall(r"LaunchCost\{\{([^}]*)\}, \{([^}]*)\}", body[:body.index(";")])
    names = "start wg tile crowd few cut fold ahead lag".split()
    kinds = [(128, True), (128, False), (64, True), (64, False)]
    return {(*kind, rows): dict(zip(names, (float(x.strip().rstrip("f")) for x in part.split(","))))
            for kind, parts in zip(kinds, sets) for rows, part in zip((128, 256), parts)}


def time_of(c, Nq, rows, units, counts):
    """Time of a launch whose units (tiles) are cut into `counts` pieces, by the model; None: it does not fit, or a piece is empty."""
    m, workgroups, slowest = -(-Nq // rows), sum(counts) * -(-Nq // rows), 0.0
    if sum(counts) > 256 // m:
        return None
    tile = c["tile"] * (1 + c["crowd"] * workgroups) * (c["few"] if 2 * Nq <= rows else 1)
    for n, k in zip(units, counts):
        length = -(-(n - int(c["ahead"]) - begin(k - 1, k, 0, int(c["lag"]))) // k)
        if k > 1 and (length < 1 or begin(k - 1, k, length, int(c["lag"])) >= n):
            return None
        slowest = max(slowest, tile * n if k == 1 else tile * length + c["cut"] + c["fold"] * (k - 1))
    return c["start"] + c["wg"] * workgroups + slowest


def test_no_cut_with_pieces_of_a_common_length_is_cheaper(b, monkeypatch):
    """Heads of up to 24 lengths, either kind of units: the cut taken costs no more by the model than any other of its kind, from whole units
    of the head with the most keys on.  (Choosing takes single precision: 1e-5 allows for sums of ten roundings of 2^-24.)"""
    rng, costs = random.Random(3), launch_costs()
    for _ in range(150):
        H, d, score, rows = rng.choice([1, 3, 12, 24]), rng.choice([64, 128]), rng.random() < 0.3, rng.choice([128, 256])
        Nq, Nc = rng.choice([1, 64, 300, 1170]), rng.choice([64, 300, 1170])
        lens = [rng.randrange(64) * rng.choice([16, 97]) for _ in range(H)]
        sinks = [rng.choice([0, n // 3]) for n in lens]
        monkeypatch.setenv("DF_ATTN_CUT", str(rows))
        got, pieces = b.df_attn_units(d, score, Nq, Nc, lens, sinks)
        units = [tiles(s) + tiles(n - s) + tiles(Nc) for n, s in zip(lens, sinks)]
        c, best = costs[d, score, rows], None
        ahead, lag = SHAPE[d, score, rows]
        assert (c["ahead"], c["lag"]) == (ahead, lag)
        for longest in range(max(1, units[lens.index(max(lens))] - ahead), 0, -1):
            counts = []
            for n in units:
                k = 1
                while k <= 256 and begin(k - 1, k, longest, lag) + longest + ahead < n:
                    k += 1
                counts.append(k)
            t = time_of(c, Nq, rows, units, counts)
            best = t if best is None or (t is not None and t < best) else best
        assert got == (rows if best is not None else 0)
        if got:
            assert time_of(c, Nq, rows, units, pieces) <= best * (1 + 1e-5), (H, d, score, rows, Nq, Nc, lens, sinks, pieces)


def test_many_lengths_take_little_longer_to_plan(b):
    """Twenty-four heads of 24 lengths against 24 of one: less than four times the host time (1.8 times here; 6.7 with a walk over
    all heads for every length of piece that is tried)."""
    rng = random.Random(24)
    rows, pieces = ctypes.c_int32(), (ctypes.c_int32 * 24)()

    def host_time(lens):
        array, best = b._i32(lens), []
        for Nq in (100, 260, 390, 700):
            args = (24, 128, 0, Nq, 200, array, None, ctypes.byref(rows), pieces)
            runs = []
            for _ in range(50):
                t = time.perf_counter()
                b.lib.df_attn_units(*args)
                runs.append(time.perf_counter() - t)
            best.append(min(runs))
        return sum(best)

    lengths = [100 + 64 * i for i in range(24)]
    one, many = host_time([800] * 24), host_time(rng.sample(lengths, 24))
    print(f"{one * 2.5e5:.1f} us, {many * 2.5e5:.1f} us")
    assert many < 4 * one


def test_long_launches_keep_their_spans(b):
    for Nq, lens, sinks in ((4680, [9360] * 9 + [0] * 3, [1560] * 9 + [0] * 3), (10800, [43200] * 12, [3600] * 12), (1170, [32760] * 12, [1560] * 12)):
        for d in (64, 128):
            for score in (False, True):
                assert b.df_attn_units(d, score, Nq, Nq, lens, sinks) == (0, [0] * 12)


def test_argument_validation(b):
    for bad, code in (((96, False, 1, 1, [0]), b.DF_ERR_UNSUPPORTED), ((64, False, 0, 1, [0]), b.DF_ERR_SHAPE),
                      ((64, False, 1, 1, [0] * 65), b.DF_ERR_UNSUPPORTED), ((128, True, 4, 4, [10], [11]), b.DF_ERR_RANGE)):
        with pytest.raises(b.DfError) as e:
            b.df_attn_units(*bad)
        assert e.value.status == code
    assert b.lib.df_attn_units(1, 64, 0, 1, 1, None, None, None, None) == b.DF_ERR_NULL

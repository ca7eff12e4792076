"""Which launches are cut unit by unit, and into what (the host's choice; no GPU)."""
import random

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

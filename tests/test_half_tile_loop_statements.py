"""The tile-loop statements for 32 keys of every tile, by the interpreter of the whole ones: group 0 takes a tile's first 32 keys,
group 1 the others, which differ in the addresses of the operands and in the key of a lane's first row."""
import io
import random

import pytest

from tests import test_tile_loop_statements as whole

TO_SECOND_HALF = 512                  # bytes from row r to row r + 32 of a tile in LDS


WAVE = whole.Wave


class BothHalves:
    """What both halves of a statement do, as the whole one would: their masks side by side (S of keys 32 to 63 lies 16 registers on)."""

    def __init__(self, statement, values, outgrown=()):
        self.halves = [WAVE(statement, dict(values, **{x: values[x] + at for x, at in shift.items()}), outgrown)
                       for shift in ({}, dict(ka=TO_SECOND_HALF, va=TO_SECOND_HALF, key0=32))]

    def run(self):
        events = []
        first, second = (x.run() for x in self.halves)
        for a, b in zip(first, second, strict=True):
            if a[0] == "read":
                assert b == (*a[:2], a[2] + TO_SECOND_HALF, a[3])
                tile_b = BothHalves.tile_bytes[a[1]]
                lds0 = dict(k=0x100, v=0x20000)[a[1]]
                assert (b[2] - lds0) // tile_b == (a[2] - lds0) // tile_b and (b[2] - lds0) % tile_b + b[3] <= tile_b
            elif a[0] != "keep":
                assert a == b
            events.append(a)
            if a[0] == "keep":
                events.append(("keep", b[1] + 16, b[2]))
        return events


@pytest.mark.parametrize("d,score", [(d, score) for d in (128, 64) for score in (False, True)])
def test_loads_and_registers_of_every_piece(monkeypatch, d, score):
    rowb, ng, _, BothHalves.tile_bytes = whole.layout(d)
    assert 32 % ng == 0 and 32 // ng * rowb == TO_SECOND_HALF
    monkeypatch.setattr(whole, "Wave", BothHalves)
    monkeypatch.setattr(whole, "reads_of", lambda d, w: 2 * (d // 32) if w == "k" else 2 * (d // 16))
    kind = f"{d}, {'true' if score else 'false'}"
    text = open(whole.INC).read().replace(f"tile_loop<{kind}, true>(", "(").replace(f"half_tile_loop<{kind}>(", f"tile_loop<{kind}, true>(")
    monkeypatch.setattr(whole, "open", lambda _: io.StringIO(text), raising=False)
    statement = whole.asm_statement(d, score, True)
    rng = random.Random(31 + d + score)
    for nt, t_begin, te in whole.pieces(rng, 60):
        outgrown = {t for t in range(t_begin, te) if rng.random() < 0.3}
        n, loads, reads, landed = whole.check_piece(d, score, True, statement, nt, t_begin, te, rng.choice([0, 1, 33, 63]),
                                                    rng.randrange(4), outgrown)
        for (group, w, tile), segment in reads.items():
            for other in range(2):
                assert landed.get((other, w, tile), n + 9) < segment, (w, tile, nt, t_begin, te)
                assert loads.get((other, w, tile + whole.NBUF), n + 9) > segment, (w, tile, nt, t_begin, te)

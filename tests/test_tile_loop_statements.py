"""The generated tile-loop statements of the attention kernel, interpreted on the CPU one wave at a time.

Scalar instructions and addresses are computed, everything else only counts as having written its result: no
instruction may read a register that is neither an input of the statement nor written by it before, or touch one that a read of
LDS is still to fill, or come too soon after what wrote it (the wait states that the generator lists).  Every load into LDS
must go through a descriptor of its head, to the byte offset and the buffer that its tile belongs to (past the descriptor's
end for a tile that the piece does not have), and the loads, waits, barriers and reads of the two groups must fit
together."""
import itertools
import os
import random
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INC = os.path.join(ROOT, "paper_2601_20499_amd", "csrc", "df_attn_phase.inc")
KT, NBUF, WAVES = 64, 4, 8
UNKNOWN = object()                    # written, value of no interest
STATEMENTS = [(d, score, live) for d in (128, 64) for score in (False, True) for live in (True, False)]


def signed(x):
    return x - (1 << 32) if x & 1 << 31 else x


def asm_statement(d, score, live):
    """Instructions (macros expanded), labels, and the operands' kinds of one statement of the include."""
    head = f"tile_loop<{d}, {'true' if score else 'false'}, {'true' if live else 'false'}>("
    lines = open(INC).read().split(head)[1].split("asm volatile(\n")[1].split("\n")
    n = next(i for i, x in enumerate(lines) if not x.strip().startswith('"'))
    code = [x.strip()[1:-1].replace("\\n", "").replace("\\t", "").replace("\\\\", "\\").replace("%=", "0") for x in lines[:n]]
    inputs, outputs, clobbers = set(), set(), set(re.findall(r'"(\w+)"', lines[n + 2]))
    for line, is_out in ((lines[n], True), (lines[n + 1], False)):
        for name, how in re.findall(r'(?:\[(\w+)\] )?"([^"]*)"\(', line):
            fixed = re.search(r"\{([sv])\[(\d+):(\d+)\]\}", how)
            regs = {f"{fixed[1]}{i}" for i in range(int(fixed[2]), int(fixed[3]) + 1)} if fixed else {name}
            if is_out:
                outputs |= regs
                # written before the last input is read
                assert "&" in how, (name, how)
            if not is_out or how.startswith("+"):
                inputs |= regs
    macros, expanded, at = {}, [], None
    for x in code:
        word = x.split()
        if word[0] == ".macro":
            at = word[1]
            macros[at] = ([w.strip(",") for w in word[2:]], [])
        elif word[0] == ".endm":
            at = None
        elif word[0] == ".purgem":
            del macros[word[1]]
        elif at:
            macros[at][1].append(x)
        elif word[0] in macros:
            params, body = macros[word[0]]
            for y in body:
                for p, v in zip(params, (w.strip(",") for w in word[1:])):
                    y = y.replace("\\" + p, v)
                expanded.append(y)
        else:
            expanded.append(x)
    assert not macros
    labels = {x[:-1]: i for i, x in enumerate(expanded) if x.endswith(":")}
    program = []
    for x in expanded:
        if x.endswith(":"):
            program.append(("label",))
            continue
        op, _, rest = x.partition(" ")
        program.append((op, *(w.strip() for w in rest.split(",") if w)))
    return program, labels, inputs, outputs, clobbers


def registers(operand):
    """Names of the registers that an operand stands for ([] for a number)."""
    operand = operand.lstrip("-")
    if operand.startswith("%["):
        return [operand[2:-1]]
    m = re.fullmatch(r"([sv])\[(\d+):(\d+)\]", operand)
    if m:
        return [f"{m[1]}{i}" for i in range(int(m[2]), int(m[3]) + 1)]
    if re.fullmatch(r"v\d+|s\d+", operand) or operand in ("vcc", "m0", "scc"):
        return [operand]
    return []


class Wave:
    """One wave's way through a statement.  Events: ("load", lds address, byte offset, descriptor words), ("wait", n),
    ("barrier",), ("read", 'k' or 'v', LDS offset, bytes), ("keep", S register, whether its key counts), ("raise",)."""

    def __init__(self, statement, values, outgrown=()):
        self.program, self.labels, inputs, self.outputs, self.clobbers = statement
        self.r = {name: values.get(name, UNKNOWN) for name in inputs}
        self.r["m0"] = UNKNOWN                       # saved and restored
        self.events, self.outgrown = [], outgrown
        self.state, self.vector = 0, False           # wait states so far; whether the instruction runs on the vector ALU
        self.wrote = {}                              # register -> (what wrote it: "mfma", "trans", "swap", other; state)
        self.in_flight = []                          # registers of the LDS reads not yet waited for

    def get(self, operand):
        regs = registers(operand)
        if not regs:
            return int(operand, 0) & 0xFFFFFFFF if re.fullmatch(r"-?(0x[0-9a-f]+|\d+)", operand) else UNKNOWN
        for x in regs:
            assert x in self.r, f"{x} is read before anything is written to it"
            self.check(x)
        return self.r[regs[0]]

    def put(self, operand, value=UNKNOWN):
        for x in registers(operand):
            assert x in self.outputs or x in self.clobbers or x == "m0", f"{x} is written but not declared"
            self.check(x)
            self.r[x] = value
            self.wrote[x] = self.kind, self.state

    def check(self, x):
        """Register x is touched by the present instruction."""
        assert not any(x in regs for regs in self.in_flight), f"{x} is touched before the read that fills it is waited for"
        kind, state = self.wrote.get(x, (None, 0))
        between = self.state - state - 1
        if self.vector and kind == "mfma" and self.kind != "mfma":
            assert between >= 8, (x, between)
        if self.vector and (kind == "trans" and self.kind != "trans"):
            assert between >= 1, (x, between)
        if kind == "swap" or self.kind == "swap" and kind or x == "vcc" and self.vector and kind:
            assert between >= 2, (x, self.kind, kind, between)
        if x == "m0" and self.kind == "load":
            assert between >= 1

    def run(self, limit=100000):
        pc, r = 0, self.r
        for _ in range(limit):
            if pc >= len(self.program):
                assert not self.in_flight
                for x, (kind, state) in self.wrote.items():       # what follows may be a vector instruction
                    assert kind != "mfma" or self.state - state >= 8, x
                return self.events
            op, *a = self.program[pc]
            pc += 1
            if op == "label":
                continue
            self.state += 1 + (int(a[0]) if op == "s_nop" else 0)
            self.vector = op[0] == "v"
            self.kind = ("mfma" if "mfma" in op else "trans" if op in ("v_exp_f32", "v_log_f32") else "swap" if "_swap_" in op else
                         "load" if op.startswith("buffer") else "other")
            if op in ("s_nop", "s_setprio"):
                continue
            if op in ("s_add_i32", "s_add_u32", "s_sub_i32", "s_mul_i32", "s_lshl_b32", "s_min_i32", "v_add_u32"):
                x, y = self.get(a[1]), self.get(a[2])
                if x is UNKNOWN or y is UNKNOWN:
                    self.put(a[0])
                else:
                    self.put(a[0], (min(signed(x), signed(y)) if op == "s_min_i32" else x << (y & 31) if op == "s_lshl_b32" else
                                    x - y if "sub" in op else x * y if "mul" in op else x + y) & 0xFFFFFFFF)
                if op[0] == "s" and "mul" not in op:
                    r["scc"] = UNKNOWN
            elif op in ("s_mov_b32", "s_movk_i32", "v_mov_b32"):
                self.put(a[0], self.get(a[1]))
            elif op == "s_mov_b64":
                src = registers(a[1])
                self.get(a[1])
                for x, y in zip(registers(a[0]), src, strict=True):
                    self.put(x, r[y])
            elif op.startswith("s_cmp_"):
                x, y = signed(self.get(a[0])), signed(self.get(a[1]))
                r["scc"] = {"lg": x != y, "eq": x == y, "ge": x >= y, "lt": x < y}[op[6:8]]
            elif op == "s_cselect_b32":
                self.put(a[0], self.get(a[1]) if r["scc"] else self.get(a[2]))
            elif op == "s_cbranch_scc1":
                assert r["scc"] is not UNKNOWN
                pc = self.labels[a[0]] if r["scc"] else pc
            elif op == "s_branch":
                pc = self.labels[a[0]]
            elif op == "s_call_b64":
                self.put(a[0], pc)
                pc = self.labels[a[1]]
                if "raise" in a[1]:
                    self.events.append(("raise",))
            elif op == "s_setpc_b64":
                pc = self.get(a[0])
            elif op == "s_cbranch_vccnz":
                self.get("vcc")
                pc = self.labels[a[0]] if signed(r["t"]) in self.outgrown else pc
            elif op == "s_waitcnt":
                if a[0].startswith("vmcnt"):
                    self.events.append(("wait", int(a[0][6:-1])))
                else:
                    left = int(re.fullmatch(r"lgkmcnt\((\d+)\)", a[0])[1])
                    self.in_flight = self.in_flight[len(self.in_flight) - left:] if left else []
            elif op == "s_barrier":
                self.events.append(("barrier",))
            elif op == "buffer_load_dwordx4":
                rsrc = registers(a[1])
                self.get(a[1])
                self.events.append(("load", self.get("m0"), self.get(a[0]), tuple(r[x] for x in rsrc)))
            elif op.startswith("ds_read"):
                addr, _, offset = a[1].partition(" offset:")
                base = self.get(addr)
                self.put(a[0])
                self.in_flight.append(registers(a[0]))
                self.events.append(("read", addr[2], base + sum(int(x) for x in offset.split("+")), 16 if "b128" in op else 8))
            elif op == "v_cmp_gt_i32":
                self.put("vcc", signed(self.get(a[1])) > signed(self.get(a[2])))
            elif op == "v_cndmask_b32":
                for x in a[1:]:
                    self.get(x)
                self.put(a[0])
                self.events.append(("keep", int(a[0][1:]), r["vcc"]))
            elif "_swap_" in op:
                for x in a:
                    self.get(x)
                    self.put(x)
            else:
                assert op.split("_")[0] == "v", op
                for x in a[1:]:
                    self.get(x)
                self.put(a[0])
        raise AssertionError("the statement does not end")


def layout(d):
    rowb = 2 * d
    ng = KT // (1024 // rowb)
    return rowb, ng, dict(k=1040, v=1056), dict(k=ng * 1040, v=ng * 1056)


def check_piece(d, score, live, statement, nt, t_begin, te, ragged, quarter, outgrown=()):
    """One piece on both groups; returns what the two groups did per segment between barriers."""
    rowb, ng, gs, tile_b = layout(d)
    nt0, nt1, nt2 = nt
    sink, win, nc = (max(0, KT * n - (ragged if n else 0)) for n in nt)
    cs = 3 * rowb + 48
    kinds = "k" if score else "kv"
    # descriptors: base (two words), size, format; all words of a head's four descriptors are told apart
    desc = {w + x: (1000 * (i + 1), i + 1, (sink + win) * rowb if x == "h" else (nc - 1) * cs + rowb, 0x00020000)
            for i, (w, x) in enumerate(itertools.product("kv", "hc"))}
    lds0 = dict(k=0x100, v=0x20000)
    lane_h, lane_c = 7 * ng * rowb + 16, 7 * ng * cs + 16          # some lane's bytes
    read0 = dict(k=0x100 + 48, v=0x20000 + 40)
    key0 = (2, 0, 8, 10)[quarter]                                    # key of a quarter's first row of a block
    values = dict(t=t_begin, te=te, nt0=nt0, nt1=nt0 + nt1, sink=sink, win=win, nc=nc, cs=cs, ldsk=lds0["k"], ldsv=lds0["v"],
                  offh=lane_h, offc=lane_c, ka=read0["k"], va=read0["v"], key0=key0)
    for i, (w, x) in enumerate((w, x) for w in "kv" for x in "hc"):
        for word in range(4):
            values[f"s{64 + 4 * i + word}"] = desc[w + x][word]

    def offset_of(t):                                               # region, byte offset of the lane in tile t
        if t >= te:
            return None, 0x7FF00000
        if t < nt0 + nt1:
            return "h", lane_h + (KT * t if t < nt0 else sink + KT * (t - nt0)) * rowb
        return "c", lane_c + KT * (t - nt0 - nt1) * cs

    n, per_tile = te - t_begin, ng // WAVES
    loads, reads, landed_at = {}, {}, {}
    for group in range(2):
        events = Wave(statement, dict(values, grp=group), outgrown).run()
        # the prologue's loads in flight: K(0), K(1), V(0), K(2), V(1), of which K(0) is waited for
        order = [("k", 0), ("k", 1), ("v", 0), ("k", 2), ("v", 1)]
        flight = [x for x in order if x[0] in kinds for _ in range(per_tile)]
        landed, segment, phase = {}, 0, 0
        issued = {w: 0 for w in kinds}

        def wait(left):
            while len(flight) > left:
                w, tile = flight.pop(0)
                landed[w, tile] = landed.get((w, tile), 0) + 1
                if landed[w, tile] == per_tile:
                    landed_at[group, w, tile] = segment             # before the barrier that ends this segment

        segment = -1
        wait(2 * per_tile * len(kinds))
        segment = 0
        phases = {w: [] for w in kinds}
        kept = {}
        for e in events:
            if e[0] == "load":
                w = "v" if issued["k"] > per_tile * phase + per_tile - 1 and not score else "k"
                i = issued[w] % per_tile
                tile = phase + (3 if w == "k" else 2)
                issued[w] += 1
                region, vo = offset_of(t_begin + tile)
                assert e[3][:2] in (desc[w + "h"][:2], desc[w + "c"][:2]), (group, w, t_begin + tile, e)
                assert e[3] in (desc[w + "h"], desc[w + "c"])
                if region:
                    assert e[3] == desc[w + region]
                    assert e[2] == vo + i * WAVES * (rowb if region == "h" else cs), (group, w, t_begin + tile)
                else:
                    assert e[3][2] <= 0x7FF00000 <= e[2] < 1 << 31
                assert e[1] == lds0[w] + tile % NBUF * tile_b[w] + i * WAVES * gs[w]
                flight.append((w, tile))
                loads[group, w, tile] = segment
                if all(issued[x] == per_tile * (phase + 1) for x in kinds):
                    phase += 1
            elif e[0] == "wait":
                wait(e[1])
            elif e[0] == "barrier":
                segment += 1
            elif e[0] == "read":
                at = e[2] - lds0[e[1]]
                buf = at // tile_b[e[1]]
                assert 0 <= buf < NBUF and at % tile_b[e[1]] + e[3] <= tile_b[e[1]]
                if not phases[e[1]] or phases[e[1]][-1][0] != buf or phases[e[1]][-1][2] == reads_of(d, e[1]):
                    phases[e[1]].append([buf, segment, 0])
                phases[e[1]][-1][2] += 1
            elif e[0] == "keep":
                kept[phase, e[1]] = e[2]
        assert segment == n and phase == n                          # one barrier and one set of loads a tile
        for w in kinds:                                             # K(i) is read in MFMA phase i, V(i) in the one behind it
            reads.update({(group, w, i): i + (w == "v") for i in range(n)})
            if live:
                assert phases[w] == [[i % NBUF, reads[group, w, i], reads_of(d, w)] for i in range(n)]
        if live:
            assert events.count(("raise",)) == len([t for t in outgrown if t_begin < t < te])
            for t in range(t_begin, te):                            # keys past the end of a region
                first, rows = (0, sink) if t < nt0 else (nt0, win) if t < nt0 + nt1 else (nt0 + nt1, nc)
                valid = rows - KT * (t - first)
                for kb, qb, v in itertools.product(range(4), range(2), range(4)):
                    reg = 240 - 48 + 8 * kb + 4 * qb + v
                    counts = 16 * kb + key0 + (0, 1, 4, 5)[v] < valid
                    assert kept.get((t - t_begin, reg), True) == counts, (t, reg)
    return n, loads, reads, landed_at


def reads_of(d, w):
    return 4 * (d // 32) if w == "k" else 2 * 2 * (d // 16)


def pieces(rng, n):
    """n (or all) pieces of 1 to 3 tiles and of 4 to 6 tiles of regions of 0 to 3 tiles, and n of any length of regions of 0 to 7."""
    short, long_, longer = [], [], []
    for nt in itertools.product(range(4), range(4), (1, 2, 3)):
        for t_begin in range(sum(nt)):
            for te in range(t_begin + 1, min(sum(nt), t_begin + 6) + 1):
                (short if te - t_begin <= 3 else long_).append((nt, t_begin, te))
    for _ in range(n):
        nt = rng.randrange(8), rng.randrange(8), rng.randrange(1, 8)
        t_begin = rng.randrange(sum(nt))
        longer.append((nt, t_begin, rng.randint(t_begin + 1, sum(nt))))
    return rng.sample(short, min(n, len(short))) + rng.sample(long_, min(n, len(long_))) + longer


@pytest.mark.parametrize("d,score,live", STATEMENTS)
def test_loads_and_registers_of_every_piece(d, score, live):
    rng = random.Random(20499 + d + 2 * score + live)
    statement = asm_statement(d, score, live)
    for nt, t_begin, te in pieces(rng, 60 if live else 300):
        outgrown = {t for t in range(t_begin, te) if rng.random() < 0.3}
        n, loads, reads, landed = check_piece(d, score, live, statement, nt, t_begin, te, rng.choice([0, 1, 63]),
                                              rng.randrange(4), outgrown)
        for (group, w, tile), segment in reads.items():
            for other in range(2):
                # what both groups loaded of the tile is in LDS before the barrier behind which it is read
                assert landed.get((other, w, tile), n + 9) < segment, (w, tile, nt, t_begin, te)
                # and no load goes where it lies until a barrier after it was read
                assert loads.get((other, w, tile + NBUF), n + 9) > segment, (w, tile, nt, t_begin, te)

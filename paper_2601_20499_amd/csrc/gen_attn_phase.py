#!/usr/bin/env python3
"""Writes df_attn_phase.inc: the tile loop of the attention kernel, one asm statement per variant.

A tile iteration of a wave has two phases.

MFMA phase: S^T = K Q^T for a 64-key tile and 32 queries (4 blocks of 16 keys x D/32 k-steps x 2 blocks
of 16 queries of v_mfma_f32_16x16x32_bf16, A operand = K rows read from LDS with ds_read_b128, B operand = the
wave's Q fragments in registers) and O^T += V^T P^T of the tile before (D/16 output blocks x 2 k-steps x 2 query blocks,
A operand = V^T read from a row-major V tile with ds_read_b64_tr_b16, B operand = P^T in registers); only the first
product where only scores are wanted.  An A operand feeds the two query blocks one after the other.

Why 16x16x32: the chip lowers its clock under matrix work (1.5 to 2.1 GHz of 2.4), and per multiply-add this shape moves
half the accumulator registers of 32x32x16.  MFMAs alone on random data, all CUs: 2.17 against 1.85 PFLOP/s (2.09
against 1.77 GHz at the same cycles).  It asks for the issue port twice as often (8 of every 16 cycles instead of 8 of
32), so the phases overlap less, but the clock gives back more: a loop of this schedule without loads ran 1370 ns
a tile (2 waves per SIMD) against 1481.

VALU phase: the loads of a later tile into LDS, then P^T = 2^(c S^T - reference) in bf16 and the sums of the
unrounded values.

Half a tile (`blocks` = 2 of its 4 blocks of 16 keys; P of 32 keys): in launches of few tiles the two groups of waves have the same
queries and each takes 32 keys of every tile.  Which is in the addresses of the operands and the key of a lane's
first row, the statement is the same for both.  An iteration takes 0.9 us there where a whole tile takes 1.6.

Why asm: the LDS reads that feed the matrix core return asynchronously.  Between
the read and the s_waitcnt that covers it the destination registers must not be touched, and
the order "wait, MFMA, next read" must not change: nothing can be scheduled into an asm statement, and its registers are
fixed.  Why the whole loop: with separate MFMA and softmax blocks the compiler held the tiles in other
registers between them, copied and spilled (158 registers), or, where it did not, spent 45 scalar instructions and ten
branches a tile on the cursors; 3055 cycles a tile and workgroup against 2660 here.  1280x720 chunk and 12
cached frames, 32x32x16 with such a loop -> 16x16x32 with such a loop -> this: 2356 -> 2277 -> 2180 us; 832x480 291 ->
284 -> 272; 1920x1088 6115 -> 5915 -> 5649.  What is not the same for every tile (the ends of regions and of the
piece, a reference that has to go up) lies behind branches in two subroutines.

The statement carries its own wait states (the compiler's hazard recogniser does not look into asm):
  * an accumulator is only reused eight MFMAs later (sixteen in the second product at d = 128), with half a tile four later in the
    first product and once a tile in the second: no dependent MFMAs back to back (the three in between hold the
    matrix core for 12 passes, and what a 4-pass MFMA writes is there after 8 wait states);
  * a vector instruction keeps 8 wait states from a 4-pass MFMA whose result it reads or overwrites (mfma_phase);
  * no instruction uses the result of an exponential or logarithm issued right before it;
  * two idle cycles (s_nop 1) between a comparison and the selection that reads vcc, and around lane swaps;
  * one instruction between a write of m0 and the load into LDS that uses it.
DEPTH operands are in flight; a wait is taken per operand.

Run this script after changing the tile layout (TileLayout in df_attn.hip) or the schedule;
the include is committed and tests/test_abi.py checks that it is what this script writes.
"""
import os

KT = 64                 # keys per tile
NBUF = 4                # LDS buffers per operand
WAVES = 8
DEPTH = 4               # operands (4 registers each) in flight
STAGE0 = 256 - 4 * DEPTH
NO_TILE = 0x7FF00000    # offset beyond every buffer: the load writes zeros

# registers of the tiles: first register of a block of four
REG_P = {(ts, qb): STAGE0 - 16 + 8 * ts + 4 * qb for ts in range(2) for qb in range(2)}
REG_S = {(kb, qb): STAGE0 - 48 + 8 * kb + 4 * qb for kb in range(4) for qb in range(2)}
REG_Q = {(ks, qb): STAGE0 - 80 + 8 * ks + 4 * qb for ks in range(4) for qb in range(2)}
REG_O = {(db, qb): STAGE0 - 144 + 8 * db + 4 * qb for db in range(8) for qb in range(2)}
# buffer descriptors: history and current chunk of K and V, and the one each cursor reads through
RSRC = dict(kh=64, kc=68, vh=72, vc=76, k=80, v=84)
KEY_OF_ROW = [0, 1, 4, 5]                   # keys of a lane's four rows of a block, from its first


def quad(r):
    return f"v[{r}:{r + 3}]"


def layout(D):
    rowb = 2 * D
    rpg = 1024 // rowb
    ng = KT // rpg
    kgs, vgs = 1024 + 16, 1024 + 32
    k_row = lambda r: (r % ng) * kgs + (r // ng) * rowb
    v_row = lambda r: (r % ng) * vgs + (r // ng) * rowb
    return dict(rowb=rowb, ng=ng, kgs=kgs, vgs=vgs, ktile=ng * kgs, vtile=ng * vgs, k_row=k_row, v_row=v_row)


def mfma_phase(D, do_qk, do_pv, koff, voff, blocks):
    """A operands in issue order (the LDS reads that fetch one, the two MFMAs it feeds), DEPTH of them in flight."""
    L = layout(D)
    mfma = "v_mfma_f32_16x16x32_bf16"
    ops = []
    for ks in range(D // 32 if do_qk else 0):
        for kb in range(blocks):
            acc = [quad(REG_S[kb, qb]) for qb in range(2)]
            ops.append(([f"ds_read_b128 @, %[ka] offset:{koff}+{L['k_row'](16 * kb) + 16 * ks}"],
                        [f"{mfma} {acc[qb]}, @, {quad(REG_Q[ks, qb])}, {acc[qb] if ks else 0}" for qb in range(2)]))
    for ts in range(blocks // 2 if do_pv else 0):
        for db in range(D // 16):
            acc = [quad(REG_O[db, qb]) for qb in range(2)]
            ops.append(([f"ds_read_b64_tr_b16 @, %[va] offset:{voff}+{L['v_row'](32 * ts + r) + 32 * db}" for r in (0, 16)],
                        [f"{mfma} {acc[qb]}, @, {quad(REG_P[ts, qb])}, {acc[qb]}" for qb in range(2)]))
    lines = []
    slot = lambda i: STAGE0 + 4 * (i % DEPTH)

    def issue(i):
        if i < len(ops):
            w = 4 // len(ops[i][0])                      # registers one read fills
            for k, r in enumerate(ops[i][0]):
                lines.append(r.replace("@", f"v[{slot(i) + w * k}:{slot(i) + w * k + w - 1}]"))

    for i in range(DEPTH):
        issue(i)
    for i, (_, mfmas) in enumerate(ops):
        pending = sum(len(o[0]) for o in ops[i + 1:i + DEPTH])
        lines.append(f"s_waitcnt lgkmcnt({pending})")
        lines += [m.replace("@", quad(slot(i))) for m in mfmas]
        issue(i + DEPTH)
    # 8 idle cycles (wait states) before a vector instruction touches what the last MFMAs wrote.  With both products that
    # is O, which only the raise of a reference touches, a softmax phase later; S is long complete, and the first instruction
    # that overwrites P comes 20 later.  (16 in every phase: 1920x1088 5692 -> 5629 us without, 1280x720 2193 -> 2173.)
    return lines + (["s_nop 1"] if do_qk and do_pv else ["s_nop 7", "s_nop 1"])


def softmax(with_p, blocks):
    """P and the row sums a0, a1, in groups of four values (one S register block each), three groups in flight: scale,
    exponential, sum and pack."""
    groups = [(kb, qb) for kb in range(blocks) for qb in range(2)]
    tmp = lambda i: STAGE0 + 4 * (i % 4)
    lines = []
    for i in range(len(groups) + 2):
        if i < len(groups):
            kb, qb = groups[i]
            lines += [f"v_fma_f32 v{tmp(i) + v}, v{REG_S[kb, qb] + v}, %[c], %[nr{qb}]" for v in range(4)]
        if 1 <= i <= len(groups):
            lines += [f"v_exp_f32 v{tmp(i - 1) + v}, v{tmp(i - 1) + v}" for v in range(4)]
        if i >= 2:
            kb, qb = groups[i - 2]
            e = [f"v{tmp(i - 2) + v}" for v in range(4)]
            if kb == 0:                                  # two chains a query block, plain adds
                lines += [f"v_add_f32 %[a{qb}], {e[0]}, {e[1]}", f"v_add_f32 %[b{qb}], {e[2]}, {e[3]}"]
            else:
                lines += [f"v_add_f32 %[{'ab'[v // 2]}{qb}], %[{'ab'[v // 2]}{qb}], {e[v]}" for v in (0, 2, 1, 3)]
            if with_p:
                p = REG_P[kb // 2, qb] + 2 * (kb % 2)
                lines += [f"v_cvt_pk_bf16_f32 v{p + v}, {e[2 * v]}, {e[2 * v + 1]}" for v in range(2)]
    return lines + ["v_add_f32 %[a0], %[a0], %[b0]", "v_add_f32 %[a1], %[a1], %[b1]"]


def raise_reference(D, with_o, blocks):
    """Subroutine: the references go up to the row's maximum so far, or to the size of its sum; l, the region sums and O
    follow.  Finite also where every key so far scores minus infinity: P of such a tile is then zero, not the NaN of
    inf - inf, and the first key that scores anything takes the reference up here again.  At a piece's first tile there is
    nothing yet that could follow."""
    t = [[f"v{STAGE0 + 4 * qb + i}" for i in range(4)] for qb in range(2)]
    lab = lambda name: f".Ldf_{name}_%="

    def over_quad(x, y, op):                             # over the four lanes that share a query
        lines = []
        for swap in ("v_permlane32_swap_b32", "v_permlane16_swap_b32"):
            lines += [f"v_mov_b32 {y}, {x}", "s_nop 1", f"{swap} {x}, {y}", "s_nop 1", f"{op} {x}, {x}, {y}"]
        return lines

    lines = [f"{lab('raise')}:"]
    for qb in range(2):
        s = [f"v{REG_S[kb, qb] + v}" for kb in range(blocks) for v in range(4)]
        m, y, sum_, alpha = t[qb]
        lines.append(f"v_max3_f32 {m}, {s[0]}, {s[1]}, {s[2]}")
        lines += [f"v_max3_f32 {m}, {m}, {s[i]}, {s[i + 1]}" for i in range(3, len(s) - 1, 2)]
        lines.append(f"v_max_f32 {m}, {m}, {s[-1]}")
        lines += over_quad(m, y, "v_max_f32")
        lines.append(f"v_mov_b32 {sum_}, %[l{qb}]")
        lines += over_quad(sum_, y, "v_add_f32")
        lines += [f"v_log_f32 {sum_}, {sum_}",
                  f"v_mul_f32 {m}, %[c], {m}",
                  "s_nop 0",
                  f"v_sub_f32 {sum_}, {sum_}, %[nr{qb}]",
                  f"v_max3_f32 {m}, {m}, {sum_}, -%[nr{qb}]",
                  f"v_max_f32 {m}, 0xff7fffff, {m}",
                  f"v_add_f32_e64 {alpha}, -%[nr{qb}], -{m}",
                  f"v_exp_f32 {alpha}, {alpha}",
                  f"v_mul_f32 %[nr{qb}], -1.0, {m}"]
    lines += ["s_cmp_lt_i32 %[again], 0",                # scc: first tile
              "s_mov_b32 %[again], %[t]",
              f"s_cbranch_scc1 {lab('raised')}"]
    for qb in range(2):
        regs = [f"%[l{qb}]", f"%[ls{qb}]", f"%[lh{qb}]"]
        if with_o:
            regs += [f"v{REG_O[db, qb] + v}" for db in range(D // 16) for v in range(4)]
        lines += [f"v_mul_f32 {r}, {r}, {t[qb][3]}" for r in regs]
    return lines + [f"{lab('raised')}:", "s_setpc_b64 %[ret]"]


def locate(D, which, ahead):
    """Cursor `which` (k or v) onto tile t + ahead: byte offset, bytes per tile, bytes between row groups, descriptor.  All
    four also for an absent tile: its loads write zeros because the offset lies past the end that a descriptor states, and
    at a piece's first tile, where K is absent in pieces of up to three tiles and V in those of up to two, no
    descriptor has been set before."""
    rowb = layout(D)["rowb"]
    lab = lambda name: f".Ldf_{name}_{which}_%="

    def through(region):
        return [f"s_mov_b64 s[{RSRC[which] + i}:{RSRC[which] + i + 1}], s[{RSRC[which + region] + i}:{RSRC[which + region] + i + 1}]"
                for i in (0, 2)]

    crosses = []
    for end in ("nt0", "nt1", "te"):
        crosses += [f"s_cmp_eq_u32 %[x0], %[{end}]", f"s_cbranch_scc1 {lab('move')}"]
    return [f"s_add_i32 %[x0], %[t], {ahead}",
            *crosses,
            "s_cmp_ge_i32 %[first], 0",                  # not the first tile, nor one where a region begins: it goes on
            f"s_cbranch_scc1 {lab('there')}",
            f"{lab('move')}:",
            "s_cmp_ge_i32 %[x0], %[te]",
            f"s_cbranch_scc1 {lab('absent')}",
            "s_cmp_ge_i32 %[x0], %[nt1]",
            f"s_cbranch_scc1 {lab('cur')}",
            "s_sub_i32 %[x1], %[x0], %[nt0]",            # sink region: row 64 t; window: sink + 64 (t - nt0)
            "s_lshl_b32 %[x1], %[x1], 6",
            "s_add_i32 %[x1], %[x1], %[sink]",
            "s_lshl_b32 %[x2], %[x0], 6",
            "s_cmp_lt_i32 %[x0], %[nt0]",
            "s_cselect_b32 %[x1], %[x2], %[x1]",
            f"s_lshl_b32 %[x1], %[x1], {rowb.bit_length() - 1}",
            f"v_add_u32 %[vo{which}], %[x1], %[offh]",
            f"s_movk_i32 %[st{which}], {KT * rowb}",
            f"s_movk_i32 %[sg{which}], {WAVES * rowb}",
            *through("h"),
            f"s_branch {lab('there')}",
            f"{lab('cur')}:",
            "s_sub_i32 %[x1], %[x0], %[nt1]",
            "s_lshl_b32 %[x1], %[x1], 6",
            "s_mul_i32 %[x1], %[x1], %[cs]",
            f"v_add_u32 %[vo{which}], %[x1], %[offc]",
            f"s_lshl_b32 %[st{which}], %[cs], 6",
            f"s_lshl_b32 %[sg{which}], %[cs], {WAVES.bit_length() - 1}",
            *through("c"),
            f"s_branch {lab('there')}",
            f"{lab('absent')}:",
            f"v_mov_b32 %[vo{which}], 0x{NO_TILE:x}",
            f"s_mov_b32 %[st{which}], 0",
            f"s_mov_b32 %[sg{which}], 0",
            *through("h"),
            f"{lab('there')}:"]


def special(D, score, live, blocks):
    """Subroutine: what is not the same for every tile, from three tiles before a boundary (of a region or the piece) on."""
    lab = lambda name: f".Ldf_{name}_%="
    lines = [f"{lab('special')}:",
             "s_cmp_lg_u32 %[t], %[bd]",
             f"s_cbranch_scc1 {lab('inside')}"]
    if live:                                             # a region ended with the tile before: what it has summed so far
        for end, reg in (("nt0", "ls"), ("nt1", "lh")):
            lines += [f"s_cmp_lg_u32 %[t], %[{end}]", f"s_cbranch_scc1 {lab('not_' + end)}",
                      f"v_mov_b32 %[{reg}0], %[l0]", f"v_mov_b32 %[{reg}1], %[l1]", f"{lab('not_' + end)}:"]
    lines += next_boundary()
    lines += [f"{lab('inside')}:", "s_sub_i32 %[ev], %[bd], 3"]
    lines += locate(D, "k", 3)
    if not score:
        lines += locate(D, "v", 2)
    if live:                                             # keys past the end of a region, in its last tile
        lines += ["s_add_i32 %[x0], %[t], 1",
                  "s_cmp_lg_u32 %[x0], %[bd]",
                  f"s_cbranch_scc1 {lab('whole')}",
                  "s_cmp_lt_i32 %[t], %[nt1]",           # x0: keys of the region, x1: its first tile
                  "s_cselect_b32 %[x0], %[win], %[nc]",
                  "s_cselect_b32 %[x1], %[nt0], %[nt1]",
                  "s_cmp_lt_i32 %[t], %[nt0]",
                  "s_cselect_b32 %[x0], %[sink], %[x0]",
                  "s_cselect_b32 %[x1], 0, %[x1]",
                  "s_sub_i32 %[x1], %[t], %[x1]",
                  "s_lshl_b32 %[x1], %[x1], 6",
                  "s_sub_i32 %[x0], %[x0], %[x1]",       # keys in the tile
                  f"s_cmp_ge_i32 %[x0], {KT}",
                  f"s_cbranch_scc1 {lab('whole')}",
                  f"v_mov_b32 v{STAGE0}, 0xff800000"]
        for kb in range(blocks):
            for v in range(4):
                lines += [f"s_sub_i32 %[x1], %[x0], {16 * kb + KEY_OF_ROW[v]}",
                          "v_cmp_gt_i32 vcc, %[x1], %[key0]",
                          "s_nop 1"]
                lines += [f"v_cndmask_b32 v{REG_S[kb, qb] + v}, v{STAGE0}, v{REG_S[kb, qb] + v}, vcc" for qb in range(2)]
        lines.append(f"{lab('whole')}:")
    # A piece's first tile sets the references before it is scaled (with none every exponential would overflow, and the
    # tile be done twice).
    first = [f"s_cbranch_scc1 {lab('raise')}"] if live else []
    return lines + ["s_cmp_lt_i32 %[first], 0", "s_mov_b32 %[first], 0", *first, "s_setpc_b64 %[ret]"]


def next_boundary():
    """bd = the first of nt0, nt1, te (all at most te) behind tile t."""
    return ["s_cmp_lt_i32 %[t], %[nt1]", "s_cselect_b32 %[bd], %[nt1], %[te]",
            "s_cmp_lt_i32 %[t], %[nt0]", "s_cselect_b32 %[bd], %[nt0], %[bd]",
            "s_min_i32 %[bd], %[bd], %[te]"]


def loads(D, score, slot):
    """This wave's share of K(t + 3) and V(t + 2)."""
    L = layout(D)
    lines = []
    for which, gs, tile, buf in (("k", L["kgs"], L["ktile"], (slot + 3) % NBUF), ("v", L["vgs"], L["vtile"], (slot + 2) % NBUF))[:1 if score else 2]:
        r = f"s[{RSRC[which]}:{RSRC[which] + 3}]"
        for i in range(L["ng"] // WAVES):
            lines.append(f"s_add_u32 m0, %[lds{which}], {buf * tile + WAVES * i * gs}")
            lines.append(f"v_add_u32 %[tmp], %[sg{which}], %[vo{which}]" if i else "s_nop 0")
            lines.append(f"buffer_load_dwordx4 %[{'tmp' if i else 'vo' + which}], {r}, 0 offen lds")
    return lines


def tile_loop(D, score, live, blocks=4):
    L = layout(D)
    dma = L["ng"] // WAVES * (1 if score else 2)         # loads a wave issues per VALU phase
    prefer_group1 = live and (score or D == 64)          # see the loop over the groups
    lab = lambda name: f".Ldf_{name}_%="
    lines = [".macro df_mfma koff, voff"] + mfma_phase(D, True, not score, "\\\\koff", "\\\\voff", blocks) + [".endm"] if live else []
    if live:
        lines += [".macro df_softmax"] + softmax(not score, blocks) + [".endm"]
        for r, init in (("l", 0), ("ls", 0), ("lh", 0), ("nr", "0x7f800000")):
            lines += [f"v_mov_b32 %[{r}{qb}], {init}" for qb in range(2)]
        if not score:
            lines += [f"v_mov_b32 v{REG_O[db, qb] + v}, 0" for db in range(D // 16) for qb in range(2) for v in range(4)]
        lines.append("s_mov_b32 %[again], -1")
    lines.append("s_mov_b32 %[first], -1")
    lines += next_boundary()
    lines.append("s_mov_b32 %[m0_was], m0")
    lines.append("s_mov_b32 %[ev], %[t]")                # the first iteration sets the cursors ...
    for which in "k" if score else "kv":                 # ... after it has moved them on like any other
        lines += [f"s_mov_b32 %[st{which}], 0", f"v_mov_b32 %[vo{which}], 0"]
    if live:
        lines += mfma_phase(D, True, False, "0", "0", blocks)
    lines += ["s_cmp_lg_u32 %[grp], 0", f"s_cbranch_scc1 {lab('group1' if prefer_group1 else 'g1_0')}"]
    for g in range(2):
        at = lambda name, slot: lab(f"{name}_g{g}_{slot}")
        # Scoring, and attention at d = 64, ask more of the issue port than of the matrix core (768 and 832 cycles a tile
        # and wave of 8 an MFMA, 8 an exponential, 4 any other instruction, against 512).  At equal priority the older
        # waves of group 0 go first in both phases and the younger ones run when these wait at the barrier: 64.9 us for
        # 832x480 sampled scores against 59.2 with group 1 first, 174 against 161 with 21 cached frames, 186.9 against
        # 167.6 for 832x480 attention at d = 64.  Attention at d = 128 (1168 against 1024) gains nothing from it, nor from
        # priority for one of the phases (under 0.3 %).
        if prefer_group1:
            lines += [f"{lab(f'group{g}')}:", f"s_setprio {2 * g}"]
        for slot in range(NBUF):
            lines.append(f"{lab(f'g{g}_{slot}')}:")
            if g == 1:
                lines += [f"s_waitcnt vmcnt({dma})", "s_barrier"]
            lines.append("v_add_u32 %[vok], %[stk], %[vok]")
            if not score:
                lines.append("v_add_u32 %[vov], %[stv], %[vov]")
            lines += ["s_cmp_ge_i32 %[t], %[ev]", f"s_cbranch_scc1 {at('call', slot)}", f"{at('ready', slot)}:"]
            lines += loads(D, score, slot)
            if live:
                lines += [f"{at('softmax', slot)}:",
                          "df_softmax",
                          "v_add_f32 %[a0], %[l0], %[a0]",
                          "v_add_f32 %[a1], %[l1], %[a1]",
                          "v_add_f32 %[tmp], %[a0], %[a1]",
                          "v_cmp_nge_f32 vcc, %[lim], %[tmp]",
                          f"s_cbranch_vccnz {at('outgrown', slot)}",
                          f"{at('summed', slot)}:",
                          "v_mov_b32 %[l0], %[a0]",
                          "v_mov_b32 %[l1], %[a1]"]
            if g == 0:
                lines += [f"s_waitcnt vmcnt({2 * dma})", "s_barrier"]
            lines += ["s_add_i32 %[t], %[t], 1", "s_cmp_eq_u32 %[t], %[te]", f"s_cbranch_scc1 {at('end', slot)}"]
            if live:
                lines.append(f"df_mfma {(slot + 1) % NBUF * L['ktile']}, {slot * L['vtile']}")
        lines.append(f"s_branch {lab(f'g{g}_0')}")
        for slot in range(NBUF):
            lines += [f"{at('call', slot)}:", f"s_call_b64 %[ret], {lab('special')}", f"s_branch {at('ready', slot)}"]
            if live:
                lines += [f"{at('outgrown', slot)}:",
                          "s_cmp_eq_u32 %[again], %[t]",       # once a tile
                          f"s_cbranch_scc1 {at('summed', slot)}",
                          f"s_call_b64 %[ret], {lab('raise')}",
                          f"s_branch {at('softmax', slot)}"]
            lines.append(f"{at('end', slot)}:")
            if live and not score and slot:
                lines.append(f"v_add_u32 %[va], {slot * L['vtile']}, %[va]")
            lines.append(f"s_branch {lab('last')}")
    if live:
        lines += raise_reference(D, not score, blocks)
    lines += special(D, score, live, blocks)
    lines.append(f"{lab('last')}:")
    if live and not score:
        lines += mfma_phase(D, False, True, "0", "0", blocks)
    lines.append("s_mov_b32 m0, %[m0_was]")
    if prefer_group1:
        lines.append("s_setprio 0")
    if live:
        lines += [".purgem df_mfma", ".purgem df_softmax"]
    return lines


def bound(how, regs, var, n):
    return [f'"{how}{{{quad(regs[i, qb])}}}"({var}[{i}][{qb}])' for i in range(n) for qb in range(2)]


def function(D, score, live, blocks=4):
    L = layout(D)
    outs = ['[t] "+&s"(t)', f'"=&{{s[{RSRC["k"]}:{RSRC["k"] + 3}]}}"(rk)', f'"=&{{s[{RSRC["v"]}:{RSRC["v"] + 3}]}}"(rv)']
    outs += [f'[{n}] "=&s"({n})' for n in ("stk", "sgk", "bd", "ev", "x0", "x1", "x2", "ret", "m0_was", "first")]
    outs += [f'[{n}] "=&v"({n})' for n in ("vok", "tmp")]
    ins = [f'[{n}] "s"(a.{n})' for n in ("te", "nt0", "nt1", "sink", "cs", "grp", "ldsk")]
    ins += [f'[{n}] "v"(a.{n})' for n in ("offh", "offc")]
    regions = ["kh", "kc"]
    if not score:
        outs += ['[stv] "=&s"(stv)', '[sgv] "=&s"(sgv)', '[vov] "=&v"(vov)']
        ins.append('[ldsv] "s"(a.ldsv)')
        regions += ["vh", "vc"]
    if live:
        outs += ['[again] "=&s"(again)'] + [f'[{n}{qb}] "=&v"({n}[{qb}])' for n in "ab" for qb in range(2)]
        outs += [f'[{n}{qb}] "=&v"(r.{f}[{qb}])' for n, f in (("l", "l"), ("ls", "l_sink"), ("lh", "l_hist"), ("nr", "neg_ref")) for qb in range(2)]
        outs += bound("=&", REG_S, "s", blocks)
        ins += [f'[{n}] "s"(a.{n})' for n in ("win", "nc", "c", "lim")] + [f'[{n}] "v"(a.{n})' for n in ("ka", "key0")]
        ins += bound("", REG_Q, "qf", D // 32)
        if not score:
            outs += ['[va] "+&v"(va)'] + bound("=&", REG_P, "pb", blocks // 2) + bound("=&", REG_O, "o", D // 16)
    ins += [f'"{{s[{RSRC[n]}:{RSRC[n] + 3}]}}"(a.{n})' for n in regions]
    clob = ['"vcc"', '"scc"', '"memory"'] + ([f'"v{r}"' for r in range(STAGE0, 256)] if live else [])
    body = "\n".join(f'        "{ln}\\n\\t"' for ln in tile_loop(D, score, live, blocks))
    name = f"tile_loop<{D}, {'true' if score else 'false'}, {'true' if live else 'false'}>"
    if blocks == 2:
        name = f"half_tile_loop<{D}, {'true' if score else 'false'}>"
    return f"""template <>
__device__ __forceinline__ void {name}(
    const TileLoopArgs &a, const bf16x8 (&qf)[{D // 32}][2], f32x4 (&o)[{D // 16}][2], RowSums &r) {{
  static_assert(TileLayout<{D}>::NG == {L['ng']} && TileLayout<{D}>::KGS == {L['kgs']} && TileLayout<{D}>::VGS == {L['vgs']} &&
                TileLayout<{D}>::ROWB == {L['rowb']} && kKT == {KT} && kNBuf == {NBUF} && kWaves == {WAVES}, "regenerate df_attn_phase.inc");
  static_assert({' && '.join(f"key_of_row({4 + v}) == {k}" for v, k in enumerate(KEY_OF_ROW))}, "the statement masks the keys {KEY_OF_ROW}");
  u32x4 rk, rv;
  int t = a.t_begin, bd, ev, again, x0, x1, x2, m0_was, first;
  unsigned stk, sgk, stv, sgv, vok, vov, tmp, va = a.va;
  unsigned long long ret;
  float a_[2], b_[2];
  f32x4 s[{blocks}][2];
  bf16x8 pb[{blocks // 2}][2];
  asm volatile(
{body}
        : {', '.join(x.replace('(a[', '(a_[').replace('(b[', '(b_[') for x in outs)}
        : {', '.join(ins)}
        : {', '.join(clob)});
}}
"""


def text():
    head = ("// Generated by gen_attn_phase.py - do not edit; see that script for the schedule and its reasons.\n"
            "// tile_loop<D, SCORE_ONLY, LIVE>: all tiles of a piece; a wave that is not LIVE (its rows lie past the last query)\n"
            "// moves tiles and keeps the barriers, but computes nothing.  half_tile_loop<D, SCORE_ONLY>: the same, live, for 32 keys of\n"
            "// every tile.\n"
            f"// Staging registers v{STAGE0}..v255, {DEPTH} operands in flight.\n")
    every = [(D, score, live, 4) for D in (128, 64) for score in (False, True) for live in (True, False)]
    every += [(D, score, True, 2) for D in (128, 64) for score in (False, True)]
    return head + "\n".join(function(*x) for x in every)


OUT = os.path.join(os.path.dirname(os.path.abspath(__file__)), "df_attn_phase.inc")

if __name__ == "__main__":
    with open(OUT, "w") as f:
        f.write(text())
    print("wrote", OUT)

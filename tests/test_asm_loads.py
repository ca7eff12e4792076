"""Inline asm that reads memory through scalar registers keeps its own distance from what wrote them: a v_readlane (the compiler
keeps scalars in lanes of vector registers) needs five wait states before a vector memory instruction that reads
its result, and the compiler does not look into asm statements."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_20499_amd", "csrc")


def statements():
    """(file, instructions, scalar operands) of every asm statement of the hand-written sources."""
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"\basm\s+volatile\s*\(", text):
            body = text[m.end():text.index(";", text.index(")", m.end()))]
            parts = re.split(r"\s*(?<!:):(?!:)\s*(?=[\"\[]|$|:|\))", re.sub(r"::", ": :", body))
            code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', parts[0])).replace("\\t", "").split("\\n")
            names, n = [], 0
            for part in parts[1:3]:
                for name, how in re.findall(r'(?:\[(\w+)\]\s*)?"([^"]*)"\s*\(', part):
                    if "s" in how:
                        names.append(f"%[{name}]" if name else f"%{n}")
                    n += 1
            yield os.path.basename(path), [x.strip() for x in code if x.strip()], names


def test_the_statements_are_found():
    found = [code for _, code, names in statements() if names and any(x.startswith("global_load") for x in code)]
    assert len(found) == 3 and {len(c) > 8 for c in found} == {True}


@pytest.mark.parametrize("file,code,names", list(statements()))
def test_wait_states_before_a_scalar_base_is_read(file, code, names):
    states = 0
    for x in code:
        if re.match(r"(global|buffer|flat)_", x) and any(re.search(re.escape(n) + r"(?!\d)", x) for n in names):
            assert states >= 5, (file, x)
            break
        states += 1 + int(x.split()[1]) if x.startswith("s_nop") else 1


def test_slots_are_loaded_behind_the_look_at_their_flag():
    """Every function that loads a whole slot either does so in one statement that clobbers memory or begins with one."""
    text = open(os.path.join(CSRC, "df_attn.hip")).read()
    bodies = re.findall(r"void (load_(?:half_)?(?:slot|stats)\w*)(?:<\d+>)?\([^;{]*\{\n(.*?)\n\}", text, flags=re.S)
    assert sorted(name for name, _ in bodies) == ["load_half_slot", "load_slot_through", "load_slot_through", "load_stats_through"]
    for name, body in bodies:
        before = body.index('"memory"')
        assert "slot_load4" not in body[:before], name

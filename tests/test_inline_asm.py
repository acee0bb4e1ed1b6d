"""The operand lists of the kernels' inline assembly, read from the sources: a block that writes m0 names
it as clobbered, and an output written before the block's last read of a separate input is early-clobber
(else the compiler may give both one register).  Host-only."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_20686_amd", "csrc")
FOLD = re.compile(r'ODGS_FOLD\((\w+), (\w+), "(\w+)", "(\w+)"\)')


def _expand(src):
    """ODGS_FOLD(D, S, CTRL, BANKS): one bank-masked DPP add."""
    return FOLD.sub(r'"v_add_f32_dpp %\1, %\2, %\2 \3 row_mask:0xf bank_mask:\4\\n"', src)


def _split(text, sep):
    """Split at `sep` outside strings and brackets."""
    parts, depth, quoted, cur = [], 0, False, ""
    for i, ch in enumerate(text):
        if ch == '"' and text[i - 1] != "\\":
            quoted = not quoted
        if not quoted:
            depth += ch in "([{"
            depth -= ch in ")]}"
        if ch == sep and depth == 0 and not quoted:
            parts.append(cur)
            cur = ""
        else:
            cur += ch
    return parts + [cur]


def asm_blocks():
    """(file, line, instructions, output constraints, input constraints, clobbers) of every asm statement."""
    out = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        src = _expand(open(path).read())
        for m in re.finditer(r"\basm(?:\s+volatile)?\s*\(", src):
            depth, end, quoted = 1, m.end(), False
            while depth:
                ch = src[end]
                quoted ^= ch == '"'
                if not quoted:
                    depth += (ch == "(") - (ch == ")")
                end += 1
            fields = (_split(src[m.end():end - 1], ":") + ["", "", ""])[:4]
            text = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', fields[0])).replace("\\t", " ")
            constraints = [[re.search(r'"([^"]*)"', op).group(1) for op in _split(f, ",") if '"' in op] for f in fields[1:]]
            out.append((os.path.basename(path), src.count("\n", 0, m.start()) + 1,
                        [line.strip() for line in text.split("\\n") if line.strip()], *constraints))
    return out


BLOCKS = asm_blocks()


def test_blocks_are_found():
    assert {"wave.h", "render.hip", "render_sph.hip"} <= {b[0] for b in BLOCKS}
    assert max(len(b[2]) for b in BLOCKS) > 20  # the thirteen-value folds


@pytest.mark.parametrize("block", BLOCKS, ids=lambda b: "%s:%d" % b[:2])
def test_operands(block):
    _, _, lines, outputs, inputs, clobbers = block
    written = {}   # output operand -> first instruction that writes it
    last_read = -1  # last instruction that reads a separate input
    for at, line in enumerate(lines):
        name, _, rest = line.partition(" ")
        ops = [o.strip().split(" ")[0] for o in rest.split(",")]
        dest = [] if name.startswith(("s_cmp", "s_nop", "s_wait")) else ops[:1]
        if "m0" in dest:
            assert "m0" in clobbers, line
        for op in ops[len(dest):]:
            if re.fullmatch(r"%\d+", op) and int(op[1:]) >= len(outputs):
                last_read = at
        for op in dest:
            if re.fullmatch(r"%\d+", op):
                assert int(op[1:]) < len(outputs), line
                written.setdefault(int(op[1:]), at)
    for op, at in written.items():
        assert "&" in outputs[op] or at >= last_read, "output %d is written before the last input is read" % op

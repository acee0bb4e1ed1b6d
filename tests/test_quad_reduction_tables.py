"""Where the bank-masked folds of the reverse compositors leave each value's partial sums in a 16-lane row,
against where their flushes read them: the fold instructions are taken from the sources and run on a model
of the DPP patterns (row_mirror: 15-i; row_half_mirror: (i & 8) | (7 - (i & 7)); bank b: lanes 4b to 4b+3).
Host-only."""
import os
import re

import numpy as np

from tests.test_inline_asm import BLOCKS, CSRC
from tests.test_row_reduction_tables import PARTNER, _const

CTRL = {"row_mirror": PARTNER["mirror"], "row_half_mirror": PARTNER["half_mirror"]}


def _folded(fname, nregs, order):
    """Registers after the fold block of a file, from random integers; `order[k]`: the register of operand k."""
    (lines,) = [b[2] for b in BLOCKS if b[0] == fname and sum("_dpp" in line for line in b[2]) > 10]
    g = np.random.default_rng(nregs).integers(0, 10**6, size=(nregs, 16))
    reg = {k: g[order[k]].copy() for k in range(nregs)}
    for line in lines:
        m = re.fullmatch(r"v_add_f32_dpp %(\d+), %(\d+), %(\d+) (\w+) row_mask:0xf bank_mask:0x([0-9a-f])", line)
        if not m:
            assert line.startswith("s_nop")
            continue
        d, a, b = (int(x) for x in m.group(1, 2, 3))
        moved = reg[a][[CTRL[m.group(4)](i) for i in range(16)]]
        banks = np.array([int(m.group(5), 16) >> (i // 4) & 1 for i in range(16)], bool)
        reg[d] = np.where(banks, moved + reg[b], reg[d])
    return g.sum(axis=1), {order[k]: v for k, v in reg.items()}


def test_nine_values():
    total, reg = _folded("render.hip", 9, [0, 1, 2, 3, 8, 4, 5, 6, 7])
    src = open(os.path.join(CSRC, "render.hip")).read()
    # a row's words: sixteen of register 0, sixteen of register 1, the four lanes of any bank of register 8
    assert "(fq < 8 ? 16 * (fq & 1) + 4 * (fq >> 1) : 32)" in src
    assert "[i * kRingStride] = gq[0];" in src and "[i * kRingStride + 16] = gq[1];" in src
    for bank in range(4):
        words = np.concatenate([reg[0], reg[1], reg[8][4 * bank:4 * bank + 4]])
        for q in range(9):
            at = 16 * (q & 1) + 4 * (q >> 1) if q < 8 else 32
            assert words[at:at + 4].sum() == total[q], q


def test_thirteen_values():
    total, reg = _folded("render_sph.hip", 13, list(range(13)))
    table = _const("render_sph.hip", "kSphQuad")
    words = np.concatenate([reg[k] for k in (0, 2, 4, 6)])
    for q in range(13):
        at = 4 * (table >> (4 * q) & 0xF)
        assert words[at:at + 4].sum() == total[q], q

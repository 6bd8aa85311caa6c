"""Checks of the device assembly that the build makes.

In kernels that fill the register file the compiler can move a live value to
another register at the join of a divergent branch before it restores the
execution mask: only the lanes of one side are copied, and the others read a
stale value later.  A kernel whose thread index was moved that way wrote its
results out of range.  `join_copies` finds such places: vector instructions
between the label that the lanes of a finished side jump to (the target of an
s_cbranch_execz) and the instruction that restores or flips the mask.  At such a
label nothing but the mask has anything to do.
"""
from __future__ import annotations

import re

_LABEL = re.compile(r"^([A-Za-z_.$][\w.$]*):")
_TO_JOIN = re.compile(r"s_cbranch_execz\s+(\.L\w+)")
# back to the lanes of before the branch, or over to its other side
_RESTORE = re.compile(r"s_or_b64\s+exec,\s*exec\b|s_(andn2|or)_saveexec_b64\b")
_OTHER_MASK = re.compile(r"s_\w+_saveexec\w*\b|s_\w+\s+exec\b|s_c?branch|s_endpgm")
# instructions that the mask does not apply to, or that write a mask
_SCALAR = re.compile(r"(s_|v_readlane|v_writelane|v_readfirstlane|v_cmp|v_nop)")


def _blocks(text: str):
    """(function, label, instructions) of every labelled block."""
    out, fn = [], None
    for line in text.split("\n"):
        m = _LABEL.match(line)
        if m:
            if not m.group(1).startswith(".L"):
                fn = m.group(1)
            out.append((fn, m.group(1), []))
            continue
        ins = line.split(";")[0].strip()
        if out and ins and not ins.startswith("."):
            out[-1][2].append(ins)
    return out


def join_copies(text: str):
    """(function, label, instructions) of the joins with vector instructions
    ahead of the mask's restore."""
    blocks = _blocks(text)
    joins = {m.group(1) for _, _, code in blocks for m in map(_TO_JOIN.match, code) if m}
    found = []
    for fn, label, code in blocks:
        if label not in joins:
            continue
        ahead = []
        for ins in code:
            if _RESTORE.match(ins):
                if ahead:
                    found.append((fn, label, ahead))
                break
            if _OTHER_MASK.match(ins):
                break
            if not _SCALAR.match(ins):
                ahead.append(ins)
    return found


def divergent_loops(text: str):
    """Functions with a loop that the lanes leave one by one, and how many."""
    out = {}
    for fn, _, code in _blocks(text):
        n = sum(bool(re.match(r"s_andn2_b64\s+exec,\s*exec\b", ins)) for ins in code)
        if n:
            out[fn] = out.get(fn, 0) + n
    return out

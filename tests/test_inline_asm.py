"""Inline assembly in the kernels declares what it uses and changes: a load to LDS, which takes its base from m0, has it
as an operand or sets it, a block that sets m0 names it as clobbered (the compiler may keep a value of its own
there across the block), one with a barrier names memory."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_03622_amd", "csrc")


def _blocks():
    for path in sorted(glob.glob(os.path.join(CSRC, "**", "*"), recursive=True)):
        if path.endswith((".hip", ".hpp", ".cpp")):
            for m in re.finditer(r"\basm\s+volatile\s*\((.*?)\);", open(path).read(), re.S):
                yield os.path.relpath(path, CSRC), m.group(1)


def test_asm_blocks_declare_their_clobbers():
    blocks = list(_blocks())
    assert blocks
    for path, body in blocks:
        template = "".join(re.findall(r'"([^"]*)"', body.split("::")[0]))
        clobbers = re.findall(r'"([^"]*)"', body.rsplit(":", 1)[1])
        sets_m0 = re.search(r"\bm0\s*,", template)
        if sets_m0:
            assert "m0" in clobbers, (path, body)
        if re.search(r"\blds\b", template):
            assert sets_m0 or '"{m0}"' in body, (path, body)
        if "s_barrier" in template:
            assert "memory" in clobbers, (path, body)

"""Inline assembly in the kernels declares what it changes: a block that writes m0 names it as clobbered (the
compiler may keep a value of its own there across the block), one with a barrier names memory."""
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
        if re.search(r"\bm0\s*,", template):
            assert "m0" in clobbers, (path, body)
        if "s_barrier" in template:
            assert "memory" in clobbers, (path, body)

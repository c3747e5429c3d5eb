"""CPU source check of the kernels' inline asm.  gfx950 needs wait states
between vector instructions that pass a value through a scalar register or to
a v_readlane / v_readfirstlane; the compiler keeps them for its own
instructions, not around ours.  So asm neither reads lanes nor takes or gives
a scalar register, but for one compare whose result only a scalar branch
uses (the scalar unit waits by itself)."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1909_10690_amd", "csrc")


def test_no_cross_lane_or_scalar_operands():
    compares = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"\basm\s*(?:volatile)?\s*\(", text):
            depth, end = 1, m.end()
            while depth:
                depth += {"(": 1, ")": -1}.get(text[end], 0)
                end += 1
            body = text[m.end():end]
            assert "readlane" not in body and "readfirstlane" not in body and "writelane" not in body, (path, body)
            if re.search(r'"[=+]?&?s"', body):
                assert "v_cmp_gt_u16_e64" in body and body.count('"=s"') == 1 and '"s"' not in body, (path, body)
                compares += 1
    assert compares == 1
    sweep = open(os.path.join(CSRC, "sweep.h")).read()
    uses = re.findall(r"[^;{}]*\bnear_edge\b[^;{}]*[;{]", sweep)
    assert all("asm(" in u or "uint64_t near_edge;" in u or "if (near_edge != 0)" in u for u in uses), uses

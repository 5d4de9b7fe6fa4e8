"""The compiler cannot see into an inline-assembly statement, so it adds no wait states
inside or behind one.  Only instructions whose hazards the sources cover themselves may
stand in one: matrix instructions with their wait states, the codes converter, register
moves.  Comparisons, carries and other instructions that pass values through scalar
registers (two wait states between a vector write and a vector read) may not."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_10531_amd", "csrc")
ALLOWED = {"s_nop", "v_mfma_f32_16x16x32_bf16", "v_cvt_scalef32_pk_bf16_fp4", "v_accvgpr_read_b32", "v_mov_b32"}


def test_inline_assembly_uses_only_covered_instructions():
    seen = set()
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for g in re.finditer(r"\basm\b\s*(?:volatile)?\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", text):
            body = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", g[1])).replace("\\n", "\n").replace("\\t", " ")
            for line in body.split("\n"):
                if not line.strip():
                    continue
                name = line.split()[0]
                assert name in ALLOWED and "vcc" not in line, "%s: %s" % (os.path.basename(path), line.strip())
                seen.add(name)
    assert seen == ALLOWED

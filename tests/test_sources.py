"""What the kernels' sources may hold (no GPU, nothing is compiled)."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2403_05527_amd", "csrc")


def asm_templates(text):
    """The template of every asm statement."""
    text = re.sub(r"//[^\n]*|/\*.*?\*/", " ", text, flags=re.S)
    found = re.findall(r"\b(?:asm|__asm__)\b\s*(?:volatile|__volatile__)?\s*\(\s*((?:\"(?:[^\"\\]|\\.)*\"\s*)+)", text)
    assert len(found) == len(re.findall(r"\b(?:asm|__asm__|__asm)\b", text)), "an asm statement that this test cannot read"
    return ["".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", t)) for t in found]


def test_inline_asm_holds_waits_and_barriers_only():
    """The compiler counts the wait states that the matrix instructions need around other instructions, but not around those in an
    asm statement, which it does not know: an instruction there that writes or reads a vector register may reach a matrix
    instruction too early, in either direction."""
    templates = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            templates += [(os.path.basename(path), t) for t in asm_templates(f.read())]
    assert templates
    for name, t in templates:
        for line in re.split(r"\\n|\\t|;", t):
            op = line.strip().split(" ")[0]
            assert op in ("", "s_waitcnt", "s_barrier"), (name, t)

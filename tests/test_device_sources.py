"""Rules that the device sources keep, checked on their text (no GPU, no compiler)."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_07590_amd", "csrc")


def test_no_instruction_is_written_in_inline_assembly():
    """The compiler knows no hazards of instructions inside an asm statement: it inserts no wait between a matrix product
    and one that reads its result.  Statements without instructions (a value kept alive, or hidden) are harmless."""
    found = []
    sources = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h")))
    assert len(sources) > 10
    for path in sources:
        text = re.sub(r"//[^\n]*|/\*.*?\*/", "", open(path).read(), flags=re.S)
        for m in re.finditer(r"\b(?:__)?asm(?:__)?\b\s*(?:volatile\b|__volatile__\b)?\s*\(\s*((?:\"(?:[^\"\\]|\\.)*\"\s*)*)", text):
            if "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1))).strip():
                found.append((os.path.basename(path), m.group(0)))
    assert not found, found

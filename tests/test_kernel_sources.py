"""Rules that the kernel sources keep and that no result shows (CPU)."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_14563_amd", "csrc")
SOURCES = sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".hpp")))


def asm_statements(text):
    """The text of each inline asm statement, up to its closing semicolon."""
    text = re.sub(r"//[^\n]*", "", text)
    return re.findall(r"\basm\b(?:\s+volatile)?\s*\(.*?\)\s*;", text, flags=re.S)


@pytest.mark.parametrize("name", SOURCES)
def test_no_lane_reads_in_inline_asm(name):
    """A lane read needs wait states after the write of its source and before a
    use of its scalar result; the compiler inserts them around instructions it
    knows, not around the text of an asm statement."""
    with open(os.path.join(CSRC, name)) as f:
        for s in asm_statements(f.read()):
            assert not re.search(r"v_(readfirstlane|readlane|writelane)", s), s

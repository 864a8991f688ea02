"""Rules of the kernel sources that no run shows."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1805_11046_amd", "csrc")


def test_inline_assembly_names_the_registers_that_it_overwrites():
    found = 0
    for path in glob.glob(os.path.join(CSRC, "*")):
        if not path.endswith((".h", ".hip", ".cpp")):
            continue
        for text in re.findall(r"\basm volatile\((.*?)\);", open(path).read(), flags=re.S):
            written = set(re.findall(r"s_mov_b32 (m0|vcc|s\d+)", text))
            clobbers = text.rpartition(":")[2]
            found += bool(written)
            for reg in written:
                assert '"%s"' % reg in clobbers, (os.path.basename(path), text)
    assert found

"""What the kernels' sources must not hold, because nothing at run time would show it reliably."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1804_10727_amd", "csrc")


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.h*"))), ids=os.path.basename)
def test_no_vector_instruction_in_inline_assembly(path):
    """The compiler keeps the distance that a read of a matrix instruction's result, a lane exchange or a scalar written by a
    vector instruction needs for its own instructions only.  Memory instructions and waits hold no such operands."""
    text = re.sub(r"//[^\n]*", "", open(path).read())
    for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(", text):
        template = re.match(r'\s*((?:"(?:[^"\\]|\\.)*"\s*)*)', text[m.end():]).group(1)
        assert not re.search(r'(?:"|\\n|\\t|\s|;)v_[a-z0-9_]+', template), f"{os.path.basename(path)}: {template.strip()}"


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.h*"))), ids=os.path.basename)
def test_wide_stores_in_inline_assembly_wait(path):
    """gfx950 wants two wait states between a store of more than eight bytes and a vector instruction that writes the registers it takes
    its data from (behind such a store of its own the compiler puts s_nop 1): the assembly has to bring them along."""
    text = re.sub(r"//[^\n]*", "", open(path).read())
    for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(", text):
        template = re.match(r'\s*((?:"(?:[^"\\]|\\.)*"\s*)*)', text[m.end():]).group(1)
        lines = [l.strip() for l in re.split(r"\\n|;", template.replace('"', "").replace("\\t", " "))]
        for i, line in enumerate(lines):
            if not re.match(r"(?:global|flat|buffer|scratch)_store_(?:dwordx[34]|b96|b128)", line):
                continue
            nop = re.match(r"s_nop (\d+)", lines[i + 1]) if i + 1 < len(lines) else None
            assert nop and int(nop.group(1)) >= 1, f"{os.path.basename(path)}: {template.strip()}"

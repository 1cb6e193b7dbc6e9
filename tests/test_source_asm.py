"""Assembly written into the kernels names every register it sets: the compiler keeps values of its own in the others."""
import re
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2210_09887_amd" / "csrc"


@pytest.mark.parametrize("path", sorted(p for p in CSRC.iterdir() if p.suffix in (".h", ".hip")), ids=lambda p: p.name)
def test_m0_is_named_where_it_is_written(path):
    for block in re.findall(r"\basm\b(?:\s+volatile)?\s*\((.*?)\);", path.read_text(), re.S):
        if re.search(r"\bs_mov_b32\s+m0\b", block):
            assert re.search(r':[^:]*"m0"', block), block

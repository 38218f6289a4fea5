"""Properties of the device sources that no result shows."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2606_18431_amd", "csrc")


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.hip"))),
                         ids=os.path.basename)
def test_inline_assembly_holds_no_instruction(path):
    """The compiler separates dependent instructions by the wait states the
    chip needs (a vector instruction after a lane read of its scalar operand
    needs two), but not where one of them is inline assembly text. Assembly
    statements here only constrain registers; an asm label names an LLVM
    intrinsic, which the compiler schedules like any other instruction."""
    src = re.sub(r"//[^\n]*|/\*.*?\*/", "", open(path).read(), flags=re.S)
    texts = re.findall(r"\b(?:__asm__|__asm|asm)\b[^(]*\(\s*((?:\"[^\"]*\"\s*)+)", src)
    assert len(texts) == len(re.findall(r"\b(?:__asm__|__asm|asm)\b", src))
    for t in texts:
        t = "".join(re.findall(r"\"([^\"]*)\"", t))
        assert t == "" or t.startswith("llvm.amdgcn."), t
